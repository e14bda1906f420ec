// moe_expert_ffn: grouped SwiGLU experts (Sec. 2.1) over the experts that the
// slot table marks as resident in the expert cache (Sec. 3.4).
//
// bf16 path: two grouped GEMMs on MFMA, both of the
// form C[rows of expert e, :] = A[rows, K] . B_s[N, K]^T with K contiguous in
// both operands:
//   up   : A = x_perm, B = the gate and up projections of slot s, interleaved
//          in 32-row groups so that one wave holds gate and up accumulators
//          for the same (row, f); the epilogue writes a = silu(g) * u as bf16;
//   down : A = a, B = the down projection of slot s; the epilogue writes bf16.
// The grid is persistent (one block per compute unit); tile t is mapped so
// that each XCD (blocks b with the same b % 8) works on a contiguous range of
// tiles: the row tiles of one expert that share a weight tile then run
// together and share it through that XCD's L2. A small prologue kernel turns
// expert_offsets and the slot table into a prefix of row tiles per resident
// expert; everything stays on the device.
// Fast path (H and F multiples of 32): `ffn_gemm_bf16_fast`, 256 x 256 x 32
// tiles, 4 waves of 128 x 128, a five-stage LDS ring filled by direct
// global->LDS DMA.
// General path (H, F multiples of 8): `ffn_gemm_bf16`, 256 x 128 x 64 tiles,
// 4 waves, register-staged LDS double buffer with zero-filled K tails.
//
// f32 path (small configurations): `ffn_f32_mfma`, float32 MFMAs; one thread per
// output element where H, F or an address does not allow 16-byte loads.
#include "common.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace moe {
namespace {

constexpr int BM = 256;
constexpr int BN = 128;
constexpr int BK = 64;
constexpr int kThreads = 256;
constexpr int kChunks = BK / 8;           // 16-byte K-chunks per tile row

// Counters after prefix[E]: 16 per-XCD tile claims (8 per GEMM), then per
// GEMM one claim counter for the split tail and kMaxTailTiles arrival
// counters (one per tail tile).
constexpr int kClaimWords = 16;
constexpr int kMaxTailTiles = 1024;
constexpr int kTailWords = 1 + kMaxTailTiles;
constexpr int kCounterWords = kClaimWords + 2 * kTailWords;

// Experts with few rows go through their own kernel (below) in items of at
// most kSmallRows rows: item = expert | chunk << 8, chunk c being the expert's
// rows kSmallRows * c on. Items with the most 16-row tiles come first, so the
// costliest units start first.
constexpr int kSmallMaxTiles = 6;
constexpr int kSmallRows = 16 * kSmallMaxTiles;
constexpr int kMaxExperts = 256;
// chunks beyond each expert's first: at most 64 rows per expert on average
constexpr int kMaxExtraItems = (64 * kMaxExperts - 1) / kSmallRows;
constexpr int kMaxItems = kMaxExperts + kMaxExtraItems;

// Rows of expert e, 0 when it is not resident; *lo: its first row.
__device__ __forceinline__ int64_t expert_rows(const int32_t* offsets, const int32_t* slot, int e,
                                               int S, int64_t max_rows, int64_t* lo_out) {
  const int s = slot ? slot[e] : e;
  int64_t lo = offsets[e], hi = offsets[e + 1];
  lo = lo < 0 ? 0 : (lo > max_rows ? max_rows : lo);
  hi = hi < lo ? lo : (hi > max_rows ? max_rows : hi);
  if (lo_out) *lo_out = lo;
  return (s < 0 || s >= S) ? 0 : hi - lo;
}

// The item list of the experts whose 16-row tile counts are in tiles[0, E)
// (LDS; 0 = not listed): every thread e < E places its expert's items at their
// rank. Returns the number of items (every thread). At most cap items are kept.
__device__ __forceinline__ int list_items(const int32_t* tiles, int E, int e, int32_t* list, int cap) {
  const int mine = e < E ? tiles[e] : 0;
  const int my_full = mine > 0 ? (mine - 1) / kSmallMaxTiles : 0;   // chunks of 6 tiles before the last
  const int my_rem = mine - my_full * kSmallMaxTiles;               // tiles of the last chunk
  int full = 0, full_before = 0, last = 0, last_before = 0;
  for (int q = 0; q < E; ++q) {
    const int t = tiles[q];
    const int f = t > 0 ? (t - 1) / kSmallMaxTiles : 0;
    const int r = t - f * kSmallMaxTiles;
    full += f;
    last += t > 0;
    full_before += q < e ? f : 0;
    last_before += r > my_rem || (r == my_rem && q < e);
  }
  if (mine > 0) {
    for (int c = 0; c < my_full; ++c)
      if (full_before + c < cap) list[full_before + c] = e | (c << 8);
    if (full + last_before < cap) list[full + last_before] = e | (my_full << 8);
  }
  return min(full + last, cap);
}

// Per-expert row-tile prefix of resident experts; also clears the counters.
// Resident experts with at most 16 * small_tiles rows (small_tiles 0 or
// kSmallMaxTiles) get no row tiles here: they are listed for the few-row
// kernel instead (small[0] = their number, small[1..] = their items).
// With split_small an expert's last row tile, when it holds at most bm / 8
// rows, is counted apart (prefix2: 0 or 1 per expert), so that the GEMMs can
// run every expert's full-cost row tiles first and these small ones last: a
// tile that short runs its K loop several times faster than the full tiles
// beside it, so kept in its column group it runs ahead of the tiles that share
// its weights in L2 and streams them from HBM alone. A last tile of more than
// bm / 8 rows keeps close enough pace to stay in place. (Both products of 6000
// Mixtral-shaped tokens: 3084 us, 3180 with bm / 16; of 2000 Qwen-shaped ones 298,
// 311 with bm / 4.)
// One thread per expert and a block scan: walked by one thread the lists took
// 12 us (60 experts) to 28 us (with 47 few-row experts) of a decode step.
__global__ void __launch_bounds__(kMaxExperts)
ffn_tiles_kernel(const int32_t* __restrict__ offsets, const int32_t* __restrict__ slot, int E,
                 int S, int64_t max_rows, int bm, int small_tiles, int split_small,
                 int32_t* __restrict__ prefix) {
  __shared__ int32_t tiles[kMaxExperts];
  __shared__ int32_t wave_run[kMaxExperts / kWave], wave_run2[kMaxExperts / kWave];
  int32_t* const small = prefix + E + 1 + kCounterWords;
  int32_t* const prefix2 = small + E + 1;
  const int e = threadIdx.x;
  int run = 0, run2 = 0;
  if (e < E) {
    const int64_t m = expert_rows(offsets, slot, e, S, max_rows, nullptr);
    const bool few = m > 0 && m <= 16 * small_tiles;
    tiles[e] = few ? (int)((m + 15) / 16) : 0;
    if (m > 0 && !few) {
      run = (int)((m + bm - 1) / bm);
      if (split_small && m - (int64_t)(run - 1) * bm <= bm / 8) {
        --run;
        run2 = 1;
      }
    }
  }
  for (int q = threadIdx.x; q < kCounterWords; q += blockDim.x) prefix[E + 1 + q] = 0;
  const int mine = run, mine2 = run2;
  for (int o = 1; o < kWave; o <<= 1) {
    const int a = __shfl_up(run, o, kWave), b = __shfl_up(run2, o, kWave);
    if (lane_id() >= o) {
      run += a;
      run2 += b;
    }
  }
  if (lane_id() == kWave - 1) {
    wave_run[e / kWave] = run;
    wave_run2[e / kWave] = run2;
  }
  __syncthreads();
  for (int w = 0; w < e / kWave; ++w) {
    run += wave_run[w];
    run2 += wave_run2[w];
  }
  if (e < E) {
    prefix[e] = run - mine;
    prefix2[e] = run2 - mine2;
  }
  if (e == E - 1) {
    prefix[E] = run;
    prefix2[E] = run2;
  }
  const int n = small_tiles > 0 ? list_items(tiles, E, e, small + 1, E) : 0;
  if (e == 0) small[0] = n;
}

// silu(g) * u with the hardware exp2 and reciprocal (about 2 ulp of float32,
// far below the bf16 rounding of the result); exp2 overflows to +inf for very
// negative g, giving g * 0 * u = -0 as the exact expression does.
__device__ __forceinline__ float swiglu(float g, float u) {
  const float e = __builtin_amdgcn_exp2f(-g * 1.4426950408889634f);
  return g * __builtin_amdgcn_rcpf(1.f + e) * u;
}

__device__ __forceinline__ int swz(int row, int chunk) {
  return chunk ^ ((row >> 1) & 7);
}

// EPI 0: SwiGLU up projection, EPI 1: down projection.
template <int EPI>
__global__ void __launch_bounds__(kThreads, 1)
ffn_gemm_bf16(const uint16_t* __restrict__ A, int64_t K,
              const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1,
              int64_t F, int64_t H,
              const int32_t* __restrict__ offsets, const int32_t* __restrict__ slot,
              int E, int64_t max_rows, const int32_t* __restrict__ prefix,
              uint16_t* __restrict__ C) {
  // EPI 0: N of the output = F (a block covers 64 f, as 64 gate + 64 up rows)
  // EPI 1: N of the output = H (a block covers 128 h)
  constexpr int kOutN = EPI == 0 ? BN / 2 : BN;
  const int64_t N_out = EPI == 0 ? F : H;
  const int64_t ldc = N_out;
  const int64_t n_tiles = (N_out + kOutN - 1) / kOutN;

  __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * BK];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BN * BK];

  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = tid / kWave;
  const int wm = wave >> 1, wn = wave & 1;

  const int64_t total = (int64_t)prefix[E] * n_tiles;
  const int64_t G = gridDim.x;               // multiple of 8
  const int64_t per_xcd = G / 8;
  const int64_t first = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;

  for (int64_t t = first; t < total; t += G) {
    // ---- decode tile -> (expert, row tile, column tile)
    int e = 0;
    while (e + 1 < E && (int64_t)prefix[e + 1] * n_tiles <= t) ++e;
    const int64_t local = t - (int64_t)prefix[e] * n_tiles;
    const int64_t me = prefix[e + 1] - prefix[e];
    const int64_t nt = local / me;
    const int64_t mt = local - nt * me;
    const int s = slot ? slot[e] : e;
    int64_t lo = offsets[e];
    lo = lo < 0 ? 0 : (lo > max_rows ? max_rows : lo);
    int64_t hi = offsets[e + 1];
    hi = hi < lo ? lo : (hi > max_rows ? max_rows : hi);
    const int64_t row0 = lo + mt * BM;
    const int64_t row_end = min(row0 + (int64_t)BM, hi);
    const int64_t n0 = nt * kOutN;

    // ---- per-thread global source pointers for the staged loads
    // A: 256 rows x 8 chunks = 2048 chunks, 8 per thread (rows tid/8 + 32 i)
    // B: 128 rows x 8 chunks = 1024 chunks, 4 per thread
    const int lrow = tid / kChunks;
    const int lch = tid % kChunks;
    const uint16_t* a_src[8];
    bool a_ok[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t r = row0 + lrow + 32 * i;
      a_ok[i] = r < row_end;
      a_src[i] = A + (a_ok[i] ? r : row0) * K + lch * 8;
    }
    const uint16_t* b_src[4];
    bool b_ok[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int n = lrow + 32 * i;          // virtual B row in the tile
      int64_t wrow;
      const uint16_t* base;
      if (EPI == 0) {
        const int grp = n >> 5;             // 32-row groups: gate, up, gate, up
        const int64_t f = n0 + (grp >> 1) * 32 + (n & 31);
        b_ok[i] = f < F;
        base = ((grp & 1) ? B1 : B0) + (int64_t)s * F * H;
        wrow = b_ok[i] ? f : 0;
      } else {
        const int64_t h = n0 + n;
        b_ok[i] = h < H;
        base = B0 + (int64_t)s * H * F;
        wrow = b_ok[i] ? h : 0;
      }
      b_src[i] = base + wrow * K + lch * 8;
    }

    f32x16_t acc[4][2];
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[mi][ni][q] = 0.f;

    uint4 ra[8], rb[4];
    auto gload = [&](int64_t k0) {
      const bool kin = k0 + lch * 8 < K;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        ra[i] = (a_ok[i] && kin) ? *reinterpret_cast<const uint4*>(a_src[i] + k0)
                                 : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        rb[i] = (b_ok[i] && kin) ? *reinterpret_cast<const uint4*>(b_src[i] + k0)
                                 : make_uint4(0, 0, 0, 0);
    };
    auto sstore = [&](int buf) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = lrow + 32 * i;
        *reinterpret_cast<uint4*>(&As[buf][r * BK + swz(r, lch) * 8]) = ra[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = lrow + 32 * i;
        *reinterpret_cast<uint4*>(&Bs[buf][r * BK + swz(r, lch) * 8]) = rb[i];
      }
    };

    const int64_t ktiles = (K + BK - 1) / BK;
    gload(0);
    sstore(0);
    __syncthreads();

    const int frow = lane & 31;         // fragment row within a 32-row MFMA tile
    const int fk = lane >> 5;           // which 8-wide half of the 16-wide K step
    for (int64_t kt = 0; kt < ktiles; ++kt) {
      const int buf = kt & 1;
      if (kt + 1 < ktiles) gload((kt + 1) * BK);
      const uint16_t* as = As[buf];
      const uint16_t* bs = Bs[buf];
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        const int ch = ks * 2 + fk;
        bf16x8_t af[4], bfr[2];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
          const int r = wm * 128 + mi * 32 + frow;
          af[mi] = *reinterpret_cast<const bf16x8_t*>(&as[r * BK + swz(r, ch) * 8]);
        }
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
          const int r = wn * 64 + ni * 32 + frow;
          bfr[ni] = *reinterpret_cast<const bf16x8_t*>(&bs[r * BK + swz(r, ch) * 8]);
        }
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
          for (int ni = 0; ni < 2; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mi], bfr[ni], acc[mi][ni], 0, 0, 0);
      }
      if (kt + 1 < ktiles) sstore(buf ^ 1);
      __syncthreads();
    }

    // ---- epilogue. 32x32 C layout: lane holds column lane % 32 and rows
    // 8 * (q / 4) + 4 * (lane / 32) + (q % 4) for q = 0..15.
    const int ccol = lane & 31;
    const int crow = (lane >> 5) * 4;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int64_t r = row0 + wm * 128 + mi * 32 + 8 * (q >> 2) + crow + (q & 3);
        if (r >= row_end) continue;
        if (EPI == 0) {
          const int64_t f = n0 + wn * 32 + ccol;
          if (f < F) {
            const float g = acc[mi][0][q];
            const float u = acc[mi][1][q];
            const float act = swiglu(g, u);
            C[r * ldc + f] = f32_to_bf16(act);
          }
        } else {
#pragma unroll
          for (int ni = 0; ni < 2; ++ni) {
            const int64_t h = n0 + wn * 64 + ni * 32 + ccol;
            if (h < H) C[r * ldc + h] = f32_to_bf16(acc[mi][ni][q]);
          }
        }
      }
    }
  }
}

// Raw buffer over `elems` 16-bit values at p.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const uint16_t* p, int64_t elems) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, (int)(uint32_t)(elems * 2),
                                           0x00027000);
}

// 16 bytes per lane of a raw buffer, from byte offset voff (lane) + soff (wave);
// past its end: zeros. NT: non-temporal.
template <bool NT>
__device__ __forceinline__ u32x4_t buf_load16(rsrc_t rs, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (int)soff, NT ? 2 : 0);
}

// ------------------------------------------------------- few rows per expert
// An expert with few rows (decode-sized batches) is bound by reading its
// weights once, not by MFMA. A block owns one unit: COLS output columns
// (weight rows) of one item of at most 96 rows. The K range is cut into four
// contiguous quarters of 32-wide steps; a wave streams one quarter of its weight
// rows through 16x16x32 MFMAs in ascending K (the rows padded to 16 * MT), and
// the four partial sums are added through LDS in quarter order: a result is the
// same whichever shape of unit computes it.
// Weights are loaded non-temporally, 8 rows x 128 bytes an instruction: whole
// cache lines. Plain streaming of 1.9 GB this way runs at 6.9 TB/s, with 16
// rows x 64 bytes, the layout the MFMA takes, at 5.2 (6.0 without the
// non-temporal hint). Two such loads hold 16 rows x 64 k; lanes l and l ^ 8
// swap one half of theirs (a row rotation by 8 under a bank mask, one
// instruction a register), which leaves two MFMA operands: lane (row r, q)
// holds the 16-byte chunk q of the row's line in the first and 4 + q in the
// second, the two K steps of the line. A quarter that begins or ends in the
// middle of a line takes that half with one 16-row x 64-byte load.
// Three shapes. kWide, 4 waves and four 16-column weight tiles a unit (32
// columns of gate and of up, or 64 of down): fewest activation loads per weight
// byte, two blocks per compute unit. kMid, the same unit with 8 waves, two of
// the tiles each, for launches of at most two row tiles whose wide units are no
// more than the compute units; with more rows the activations, which both halves
// of its waves load, cost more than the waves give (one expert of 53 rows, H
// 2048, F 5632: 49 us, 44 with kWide). kNarrow, 4 waves and one 16-column tile
// (of gate and of up, or of down), where those are no more than the compute
// units either (one expert of width 5632 has 32 wide units in its down
// projection, 128 narrow ones).
constexpr int kSmallRC = 2;                      // row tiles per LDS reduction pass

constexpr int kWide = 0, kMid = 1, kNarrow = 2;

template <int EPI, int SHAPE>
struct SmallShape {
  static constexpr int NB = EPI == 0 ? 2 : 1;    // gate and up, or down
  static constexpr int NT = SHAPE == kNarrow ? 1 : 4 / NB;   // 16-column MFMA tiles per unit
  static constexpr int COLS = 16 * NT;
  static constexpr int WAVES = SHAPE == kMid ? 8 : 4;
  static constexpr int TPW = NT * NB * 4 / WAVES;            // weight tiles per wave
};

// K blocks of 64 loaded per batch: eight weight tiles of them a wave while the
// rows are few, half of that beside the activations of more row tiles (which
// weigh most in a wave of one weight tile); no instance spills a register
template <int MT, int TPW>
constexpr int small_unroll() {
  return (MT == 1 || (MT == 2 && TPW > 1) ? 8 : MT == 2 || TPW > 1 ? 4 : 2) / TPW;
}

__device__ __forceinline__ uint32_t ror8_into(uint32_t keep, uint32_t from, bool high) {
  // lanes 8..15 (high) or 0..7 of each row of 16 take `from` of the lane 8 away
  return high ? (uint32_t)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xf, 0xc, false)
              : (uint32_t)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xf, 0x3, false);
}

// MTMAX: the most row tiles of any item the launch supports; each unit takes
// the body for its item's tile count (uniform per block).
// build: the list is made here, by every block for itself (and left in `small`
// by block 0 for the down projection), instead of coming from the tile-list
// kernel: saves that launch where nothing needs the large tiles.
template <int EPI, int MTMAX, int SHAPE>
__global__ void __launch_bounds__((64 * SmallShape<EPI, SHAPE>::WAVES)) __attribute__((amdgpu_waves_per_eu(2)))
ffn_small_bf16(const uint16_t* __restrict__ A, int64_t K, const uint16_t* __restrict__ B0,
               const uint16_t* __restrict__ B1, int64_t F, int64_t H,
               const int32_t* __restrict__ offsets, const int32_t* __restrict__ slot, int E, int S,
               int64_t max_rows, int build, int32_t* __restrict__ small,
               uint16_t* __restrict__ C) {
  using SS = SmallShape<EPI, SHAPE>;
  constexpr int NB = SS::NB, NT = SS::NT, W = SS::WAVES, TPW = SS::TPW;
  constexpr int RC = MTMAX < kSmallRC ? MTMAX : kSmallRC;
  __shared__ f32x4_t part[4][RC][NT * NB][kWave];
  __shared__ int32_t s_list[EPI == 0 ? kMaxItems : 1];
  int n_items;
  const int32_t* list = small + 1;
  if (EPI == 0 && build) {
    // the tile counts live in the reduction buffer, which is not in use yet
    int32_t* const tiles = reinterpret_cast<int32_t*>(part);
    static_assert(sizeof(part) >= kMaxExperts * 4, "tile counts");
    int n = 0;
    for (int e = threadIdx.x; e < E; e += blockDim.x)
      tiles[e] = (int)((expert_rows(offsets, slot, e, S, max_rows, nullptr) + 15) / 16);
    __syncthreads();
    // E <= 256 <= threads
    n = list_items(tiles, E, (int)threadIdx.x, s_list, kMaxItems);
    __syncthreads();
    n_items = n;
    list = s_list;
    if (blockIdx.x == 0) {
      for (int q = threadIdx.x; q < n; q += blockDim.x) small[1 + q] = s_list[q];
      if (threadIdx.x == 0) small[0] = n;
    }
  } else {
    n_items = small[0];
  }
  const int64_t N_out = EPI == 0 ? F : H;        // a multiple of 32 (fast path)
  const int ncb = (int)((N_out + SS::COLS - 1) / SS::COLS);
  const int64_t units = (int64_t)n_items * ncb;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int r = lane & 15;                       // A row / B column of this lane
  const int q4 = lane >> 4;                      // its slice of a K step
  const int quarter = wave & 3, t0 = (wave >> 2) * TPW;   // its K range and first weight tile
  const int64_t ks = K / 32;
  const int64_t per = (ks + 3) / 4;
  const int64_t kb = min(ks, quarter * per), ke = min(ks, kb + per);
  // whole lines are blocks b0 .. b1 - 1; a half line before and one after them
  const bool head = (kb & 1) != 0 && kb < ke, tail = (ke & 1) != 0 && kb < ke;
  const int64_t b0 = (kb + 1) / 2, b1 = max(b0, ke / 2);
  // byte offsets from a weight tile's first row: this lane's slice of an
  // 8-row x 128-byte load, and of a 16-row x 64-byte one
  const uint32_t b_off = (uint32_t)(((int64_t)(lane & 7) * K + (q4 + ((lane >> 3) & 1) * 4) * 8) * 2);
  const uint32_t b_off32 = (uint32_t)(((int64_t)r * K + q4 * 8) * 2);
  const uint32_t b_half = (uint32_t)(8 * K * 2);       // the tile's rows 8 to 15
  auto run_unit = [&](auto mt_c, int e, int cb, int m, int64_t lo) {
    constexpr int MT = decltype(mt_c)::value;
    constexpr int U = small_unroll<MT, TPW>();
    const int s = __builtin_amdgcn_readfirstlane(slot ? slot[e] : e);
    const int64_t n0 = (int64_t)cb * SS::COLS;
    // Raw buffers: 32-bit lane offsets, and the K position as the scalar offset,
    // where pointers would take two registers and a vector addition each (66
    // registers of the shapes of five and six row tiles were spilled). Rows past
    // m lie past the end of the buffer: nothing is read and zeros are used.
    const auto rs_a = make_rsrc(A + lo * K, m * K);
    uint32_t a_off[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) a_off[i] = (uint32_t)(((int64_t)(16 * i + r) * K + q4 * 8) * 2);
    // a column tile past N_out (the last unit of a down projection whose
    // width is an odd multiple of 32) re-reads the unit's first tile and is
    // not stored
    rsrc_t rs_b[TPW];
#pragma unroll
    for (int g = 0; g < TPW; ++g) {
      const int j = (t0 + g) / NB;
      const int64_t n = n0 + 16 * j < N_out ? n0 + 16 * j : n0;
      rs_b[g] = make_rsrc(((t0 + g) % NB == 0 ? B0 : B1) + ((int64_t)s * N_out + n) * K, 16 * K);
    }
    f32x4_t acc[MT][TPW];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int g = 0; g < TPW; ++g) acc[i][g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mfma = [&](f32x4_t& c, const u32x4_t& a, const u32x4_t& w) {
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                  __builtin_bit_cast(bf16x8_t, w), c, 0, 0, 0);
    };
    // From three row tiles on, a batch's loads go out before its products, the
    // activations first (they come from L2): left to the scheduler they sink
    // between the products and few are in flight (60 experts of 64 rows, H 2048,
    // F 1408: 330 us, in this order 289). With fewer rows it does better alone
    // (16 rows: 197 us, 206 so ordered).
    constexpr bool kMany = MT > 2;
    struct Block { u32x4_t a[2][MT], w[TPW][2]; };
    struct Half { u32x4_t a[MT], w[TPW]; };
    auto load_block = [&](Block& k, int64_t blk) {
      const uint32_t kbyte = (uint32_t)blk * 128;
      auto acts = [&]() {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) k.a[hh][i] = buf_load16<false>(rs_a, a_off[i] + hh * 64, kbyte);
      };
      if (kMany) acts();
#pragma unroll
      for (int g = 0; g < TPW; ++g)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) k.w[g][hh] = buf_load16<true>(rs_b[g], b_off, kbyte + hh * b_half);
      if (!kMany) acts();
    };
    auto use_block = [&](const Block& k) {
#pragma unroll
      for (int g = 0; g < TPW; ++g) {
        u32x4_t w0, w1;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          w0[v] = ror8_into(k.w[g][0][v], k.w[g][1][v], true);
          w1[v] = ror8_into(k.w[g][1][v], k.w[g][0][v], false);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) mfma(acc[i][g], k.a[0][i], w0);
#pragma unroll
        for (int i = 0; i < MT; ++i) mfma(acc[i][g], k.a[1][i], w1);
      }
    };
    auto load_half = [&](Half& k, int64_t step) {
#pragma unroll
      for (int g = 0; g < TPW; ++g) k.w[g] = buf_load16<true>(rs_b[g], b_off32, (uint32_t)step * 64);
#pragma unroll
      for (int i = 0; i < MT; ++i) k.a[i] = buf_load16<false>(rs_a, a_off[i], (uint32_t)step * 64);
    };
    auto use_half = [&](const Half& k) {
#pragma unroll
      for (int g = 0; g < TPW; ++g)
#pragma unroll
        for (int i = 0; i < MT; ++i) mfma(acc[i][g], k.a[i], k.w[g]);
    };
    // the blocks that do not fill a batch go with the half line: after the one
    // before them, else ahead of the one after them (all conditions are uniform)
    const int rem = (int)((b1 - b0) % U);
    auto part_batch = [&](bool before, int64_t first, int n, bool after) {
      Half h;
      Block k[U > 1 ? U - 1 : 1];
      if (before) load_half(h, kb);
#pragma unroll
      for (int u = 0; u < U - 1; ++u)
        if (u < n) load_block(k[u], first + u);
      if (after) load_half(h, ke - 1);
      if (kMany) __builtin_amdgcn_sched_barrier(0);
      if (before) use_half(h);
#pragma unroll
      for (int u = 0; u < U - 1; ++u)
        if (u < n) use_block(k[u]);
      if (after) use_half(h);
    };
    if (head) part_batch(true, b0, rem, false);
    const int64_t m0 = head ? b0 + rem : b0, m1 = head ? b1 : b1 - rem;
    for (int64_t blk = m0; blk < m1; blk += U) {
      Block k[U];
#pragma unroll
      for (int u = 0; u < U; ++u) load_block(k[u], blk + u);
      if (kMany) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) use_block(k[u]);
    }
    if (m1 < b1 || tail) part_batch(false, m1, (int)(b1 - m1), tail);
    // the quarters' partial sums, RC row tiles at a time: every wave writes its
    // own, then wave q adds up the (row tile, column tile) groups g with
    // g % W == q and stores them. C layout of the 16x16 MFMA: lane holds
    // column (lane % 16), rows 4 * (lane / 16) + q of its 16-row tile. The lane
    // number is made opaque so that addresses are formed here, not kept in
    // registers over the K loop.
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int i0 = 0; i0 < MT; i0 += RC) {
#pragma unroll
      for (int ii = 0; ii < RC; ++ii)
        if (i0 + ii < MT)
#pragma unroll
          for (int g = 0; g < TPW; ++g) part[quarter][ii][t0 + g][ln] = acc[i0 + ii][g];
      __syncthreads();
      const int groups = (MT - i0 < RC ? MT - i0 : RC) * NT;
      for (int g = wave; g < groups; g += W) {
        const int ii = g / NT, j = g % NT;
        const int64_t col = n0 + 16 * j + (ln & 15);
        f32x4_t t[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          t[b] = part[0][ii][j * NB + b][ln];
#pragma unroll
          for (int q = 1; q < 4; ++q) t[b] += part[q][ii][j * NB + b][ln];
        }
        if (col >= N_out) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int rr = 16 * (i0 + ii) + (ln >> 4) * 4 + q;
          if (rr >= m) continue;
          const float v = EPI == 0 ? swiglu(t[0][q], t[NB - 1][q]) : t[0][q];
          C[(lo + rr) * N_out + col] = f32_to_bf16(v);
        }
      }
      __syncthreads();                             // part is rewritten next
    }
  };
  // units (item, column block) in list order, the grid striding over them:
  // at any time the blocks work on neighbouring columns
  for (int64_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
    // the same for the whole block, and known to be (scalar registers)
    const int32_t it = __builtin_amdgcn_readfirstlane(list[(int)(unit / ncb)]);
    const int e = it & 255;
    const int cb = __builtin_amdgcn_readfirstlane((int)(unit % ncb));
    int64_t lo;
    const int64_t rows = expert_rows(offsets, slot, e, S, max_rows, &lo);
    const int64_t skip = (int64_t)(it >> 8) * kSmallRows;
    lo = __builtin_amdgcn_readfirstlane((int)lo) + skip;        // rows are counted in 32 bits
    // 1 .. 16 * MTMAX (the list's rule)
    const int m = __builtin_amdgcn_readfirstlane((int)min(rows - skip, (int64_t)kSmallRows));
    const int mt = (m + 15) / 16;
    if (mt <= 1) run_unit(std::integral_constant<int, 1>{}, e, cb, m, lo);
    else if (mt == 2) { if constexpr (MTMAX >= 2) run_unit(std::integral_constant<int, 2>{}, e, cb, m, lo); }
    else if (mt == 3) { if constexpr (MTMAX >= 3) run_unit(std::integral_constant<int, 3>{}, e, cb, m, lo); }
    else if (mt == 4) { if constexpr (MTMAX >= 4) run_unit(std::integral_constant<int, 4>{}, e, cb, m, lo); }
    else if (mt == 5) { if constexpr (MTMAX >= 5) run_unit(std::integral_constant<int, 5>{}, e, cb, m, lo); }
    else { if constexpr (MTMAX >= 6) run_unit(std::integral_constant<int, 6>{}, e, cb, m, lo); }
  }
}

// ------------------------------------------------------- LDS DMA helpers
typedef __attribute__((address_space(3))) void lds_void;

// 16 bytes per lane of a raw buffer into LDS, from byte offset voff (lane) + soff (wave).
__device__ __forceinline__ void buf_dma16(rsrc_t rs, uint32_t voff, uint32_t soff, void* lds_wave_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)lds_wave_base, 16, (int)voff, (int)soff, 0, 0);
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// ------------------------------------------------------- bf16 fast path
// 256 x 256 block tiles, K in steps of 32, 4 waves (one per SIMD), each
// owning a 128 x 128 quarter of the output: 8 x 8 accumulators of
// v_mfma_f32_16x16x32_bf16, 256 registers, held in the accumulation registers.
// What bounds it is power and the gaps between MFMAs. The chip lowers its clock
// under MFMA load, and a product in this shape takes less energy than in the
// 32x32x16 one, whose accumulators are read and written twice as often per
// flop: a loop of nothing but MFMAs on random data runs at 2000 against 1757
// TFLOP/s.
// Operands move from global memory straight into LDS (buffer loads of 16 bytes
// a lane: each lane deposits its bytes at M0 + 16 * lane; the row is a 32-bit
// lane offset, the K offset the scalar offset), with an XOR swizzle applied on
// the load side by choosing which K-chunk each lane fetches. A K-step takes 64
// bytes of a row, half a cache line, so K-steps are loaded in pairs: the two
// halves of a line are requested by neighbouring instructions and the second
// is served by the vector cache. Loaded one step at a time every line was
// asked of L2 twice (2.37e8 L2 reads a gate/up launch of 8 x 1024 rows, now
// 1.20e8). A ring of five LDS stages holds the pair in use, the pair that has
// landed or is landing, and a stage that lets the next pair start while the
// first stage of the pair in use is still needed by nobody: the loads of a
// pair are spread evenly over two K-steps (bunched they stall the issue of
// MFMAs) and have one more K-step to land; the weights, which come from HBM,
// go first.
// Within a K-step the upper half of the A fragments is read while the MFMAs of
// the lower half run, and the next step's B fragments and lower half of A while
// those of the upper half run, one read after each of the first MFMAs.
// Measured, both GEMMs, one launch (H 4096, F 14336): 8 experts of 1024 rows
// 2537 -> 2124 us (1137 -> 1359 TFLOP/s), of 998 to 1077 rows 2778 -> 2390 us;
// 48 experts of 410 to 12000 rows (H 2048, F 1408) 1662 -> 1466 us; MFMAs run
// in 70 to 75 % of the cycles, 60 to 62 % before.
// A tile whose expert has at most 128 rows left is computed by all 4 waves
// side by side (each 32, 64 or 128 rows x 64 columns), so a ragged last row
// tile costs in proportion to its rows, on every SIMD.
// Needs K % 32 == 0.
namespace fast {
constexpr int BM = 256, BN = 256, BK = 32, STAGES = 5;
constexpr int kWaves = 4, kThreads = kWaves * 64;
constexpr int CPR = BK / 8;                 // 16-byte chunks per tile row
constexpr int RPW = 128 / BK;               // rows per 256-byte bank window
constexpr int ROWS_PER_PIECE = 512 / BK;    // rows per 1 KB DMA piece
constexpr int PIECES = BM * BK / 512;       // 1 KB pieces per operand stage
constexpr int PPW = PIECES / kWaves;        // pieces per wave per operand
constexpr int kStage = BM * BK;             // elements per operand stage
// Split-K of the last, partial round of tiles: at most kMaxSplit pieces per
// tile, each at least kMinSplitSteps K-steps; a piece's fp32 partial tile is
// 256 threads x 64 float4 (256 KB) in the workspace. A piece pays a prologue,
// its partial tile's stores and a share of the final sum whatever its length,
// which shorter pieces do not earn back: at least 32 steps instead of 64 makes
// both products of 8192 Qwen-shaped tokens 658 us instead of 590. Against no
// split, pieces of 64 steps lose too where K has 128 (8 experts, 777 tokens, K
// 4096 and 14336: 898 us, 817 with at least 128; 16 experts, 2048 tokens, H 1024,
// F 4096: 312, 244); a longer limit would order the sums of such tiles otherwise.
constexpr int kMaxSplit = 8, kMinSplitSteps = 64;
constexpr int kMaxPieces = 512;
constexpr size_t kPieceBytes = 256 * 64 * 16;
static_assert(BM == BN, "A and B stages share the piece layout");
static_assert(STAGES * 2 * kStage * 2 <= 160 * 1024, "LDS");
// row groups g = 0..3 of RPW rows take chunk c at c ^ {0, 2, 3, 1}[g]: any 16
// lanes that a 16-byte LDS read serves together (16 rows of one chunk, or two
// groups of rows of one chunk and the other two of its neighbour) then hit
// each of the 64 banks once. Unsigned: only the row's low four bits count, and
// the compiler sees it; with signed division every fragment's address was formed
// by itself, kept over the tile loop and spilled (118 registers, now 70: both
// products of 300 rows, H 512, F 512 58 -> 53 us, 60 experts of 300 rows, H 2048,
// F 1408 453 -> 434).
__device__ __forceinline__ int swz(unsigned r, int c) {
  const int g = (r / RPW) % CPR;
  return c ^ (((g & 1) << 1) ^ ((g >> 1) * 3));
}
}  // namespace fast

// The fast path addresses 256 rows of a weight matrix or of an activation with
// 32-bit byte offsets.
inline bool fast_path(int64_t H, int64_t F) {
  return H % fast::BK == 0 && F % fast::BK == 0 && F * H < ((int64_t)1 << 31) &&
         std::max(H, F) <= ((int64_t)1 << 22);
}

// Partial tiles the workspace holds for the split tail of either GEMM.
inline int64_t max_split_pieces(int64_t max_rows, int64_t H, int64_t F, int E) {
  const int64_t row_tiles = ceil_div(max_rows, fast::BM) + E;
  const int64_t col_tiles = std::max(ceil_div(F, fast::BN / 2), ceil_div(H, fast::BN));
  return std::min<int64_t>(fast::kMaxPieces,
                           fast::kMaxSplit * std::min<int64_t>(row_tiles * col_tiles, kMaxTailTiles));
}

// Workgroup barrier for the K loop: this wave's LDS reads have returned
// (a stage is refilled by DMA only after every wave passed the barrier that
// follows its last reads) and its DMA of the awaited step was waited for
// beforehand; no memory fence, which would drain every DMA in flight. The
// asm's memory clobber keeps the compiler from moving any load or store
// (LDS reads of the next stage in particular) across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// acc += a . b, accumulated in place in the accumulation registers. Written as
// asm with the accumulator tied: with the builtin and 64 four-register
// accumulators the register allocator rotates them through copies (five
// register moves per MFMA in the K loop). The compiler does not see an MFMA
// here, so idle instructions stand between the last one and the first read of
// an accumulator, and between their clearing and the first one.
__device__ __forceinline__ void mfma_acc(f32x4_t& acc, const bf16x8_t& a, const bf16x8_t& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

template <int EPI>
__global__ void __launch_bounds__(fast::kThreads, 1)
ffn_gemm_bf16_fast(const uint16_t* __restrict__ A, int64_t K,
                 const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1,
                 int64_t F, int64_t H,
                 const int32_t* __restrict__ offsets, const int32_t* __restrict__ slot,
                 int E, int64_t max_rows, const int32_t* __restrict__ prefix,
                 const int32_t* __restrict__ prefix2,
                 int32_t* __restrict__ claim, int32_t* __restrict__ tail,
                 float* __restrict__ partial, int max_pieces, uint16_t* __restrict__ C) {
  constexpr int BM = fast::BM, BN = fast::BN, BK = fast::BK, STAGES = fast::STAGES;
  constexpr int CPR = fast::CPR, ROWS_PER_PIECE = fast::ROWS_PER_PIECE, PPW = fast::PPW;
  constexpr int kStage = fast::kStage;
  auto swz = [](int r, int c) { return fast::swz(r, c); };
  constexpr int kOutN = EPI == 0 ? BN / 2 : BN;
  const int64_t N_out = EPI == 0 ? F : H;
  const int64_t ldc = N_out;
  const int64_t n_tiles = (N_out + kOutN - 1) / kOutN;

  __shared__ __attribute__((aligned(1024))) uint16_t As0[kStage], As1[kStage], As2[kStage], As3[kStage], As4[kStage];
  __shared__ __attribute__((aligned(1024))) uint16_t Bs0[kStage], Bs1[kStage], Bs2[kStage], Bs3[kStage], Bs4[kStage];
  uint16_t* const As[STAGES] = {As0, As1, As2, As3, As4};
  uint16_t* const Bs[STAGES] = {Bs0, Bs1, Bs2, Bs3, Bs4};
  // The claim broadcast lives in the fifth A stage: it is written and read
  // between tiles, when no DMA targets that stage (a tile's prologue loads
  // stages 0 to 3, and the fifth only after a barrier of its first K-step),
  // and s_last after every wave has left the K loop.
  int64_t& s_claim = *reinterpret_cast<int64_t*>(As4);
  int& s_piece = *reinterpret_cast<int*>(As4 + 4);
  int& s_last = *reinterpret_cast<int*>(As4 + 6);

  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int frow = lane & 15;                 // fragment row within a 16-row MFMA tile
  const int fk = lane >> 4;                   // which 8-wide quarter of a K-step
  const int lrow = lane / CPR;                // row within a DMA piece
  const int lpch = lane % CPR;                // physical chunk this lane fills

  // tiles: every expert's full-cost row tiles (prefix), then the small last
  // row tiles (prefix2), each in (expert, column tile, row tile) order
  const int64_t total_big = (int64_t)prefix[E] * n_tiles;
  const int64_t total = total_big + (int64_t)prefix2[E] * n_tiles;
  if (total == 0) return;                      // every expert went to the few-row kernels
  const int64_t G = gridDim.x;                 // persistent grid, a multiple of 8
  const int64_t per_xcd = G / 8;
  // Claim chunk: an XCD's whole share of a round, or 16 consecutive tiles
  // when some expert has 8 or more full-cost row tiles (a column's row tiles
  // then fill a 32-tile chunk by themselves, one weight tile against 32
  // activation panels; 16 divides the share, so the chunks of the 8 XCDs
  // still cover each round exactly once). With at most 7 row tiles per expert
  // the larger chunk cuts fewer column groups across two XCDs' L2s. Either chunk
  // for all is now within 2 % of this (8192 Qwen-shaped tokens 590 us, 584 with
  // either; 16384 DeepSeek-shaped 1520, 1508 with 16, 1531 with 32).
  int64_t me_max = 0;
  for (int ee = 0; ee < E; ++ee) me_max = max(me_max, (int64_t)(prefix[ee + 1] - prefix[ee]));
  const int64_t chunk = me_max >= 8 && per_xcd % 16 == 0 ? 16 : per_xcd;
  const int xcd = blockIdx.x % 8;
  const int64_t ksteps = K / BK;

  // Whole rounds of G tiles are claimed per XCD (each XCD walks its own
  // chunks of consecutive tiles, so the row tiles that share a weight tile
  // run together on one L2). The last, partial round of rem tiles is
  // split along K into `split` pieces claimed from one global counter,
  // chosen to minimise ceil(rem * split / G) / split rounds.
  const int64_t full = total / G * G;
  const int64_t rem = total - full;
  int64_t split = 1;
  for (int64_t sp = 2; sp <= fast::kMaxSplit; ++sp) {
    if (ksteps / sp < fast::kMinSplitSteps || rem * sp > max_pieces) break;
    if (((rem * sp + G - 1) / G) * split < ((rem * split + G - 1) / G) * sp) split = sp;
  }

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using I4 = std::integral_constant<int, 4>;

  bool in_tail = false;                        // thread 0 only
  // thread 0: the next whole-round claim, issued while the current tile runs
  // The counter's address is made opaque so the compiler does not rewrite the
  // one-lane atomic into its wave-aggregated form, which reads the result at
  // once; this way the round trip overlaps the tile and only the next claim
  // waits for it.
  __attribute__((address_space(1))) int32_t* claim_x =
      (__attribute__((address_space(1))) int32_t*)(claim + xcd);
  asm volatile("" : "+v"(claim_x));
  int32_t j_next =
      tid == 0 ? __hip_atomic_fetch_add(claim_x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  for (;;) {
    if (tid == 0) {
      int64_t tt = -1;
      int pc = 0;
      if (!in_tail) {
        const int64_t j = j_next;
        const int64_t c = ((j / chunk) * 8 + xcd) * chunk + (j % chunk);
        if (c < full) tt = c;
        else in_tail = true;
      }
      if (in_tail) {
        const int64_t u = atomicAdd(&tail[0], 1);
        if (u < rem * split) {
          tt = full + u / split;
          pc = (int)(u % split);
        }
      }
      s_claim = tt;
      s_piece = pc;
    }
    // LDS only: the claim, and every wave's last reads of the staging stages
    // before the prologue refills them; the previous epilogue's global
    // stores drain on their own (nothing in this launch reads them)
    lds_barrier();
    const int64_t t = s_claim;
    const int piece = s_piece;
    if (t < 0) break;
    if (tid == 0 && !in_tail)
      j_next = __hip_atomic_fetch_add(claim_x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool split_tile = t >= full && split > 1;
    // pieces start at even K-steps (whole 128-byte lines)
    const int64_t kbeg = split_tile ? (piece * ksteps / split) & ~(int64_t)1 : 0;
    const int64_t kend = split_tile && piece + 1 < split ? ((piece + 1) * ksteps / split) & ~(int64_t)1 : ksteps;
    const int64_t nks = kend - kbeg;
    // the last expert whose first tile is at or before t (binary search)
    int e = 0;
    int64_t nt, mt;
    if (t < total_big) {
      for (int hi = E - 1; e < hi;) {
        const int mid = (e + hi + 1) >> 1;
        if ((int64_t)prefix[mid] * n_tiles <= t) e = mid;
        else hi = mid - 1;
      }
      const int64_t local = t - (int64_t)prefix[e] * n_tiles;
      const int64_t me = prefix[e + 1] - prefix[e];
      nt = local / me;
      mt = local - nt * me;
    } else {
      const int64_t u = t - total_big;
      const int64_t si = u / n_tiles;          // which small row tile
      for (int hi = E - 1; e < hi;) {
        const int mid = (e + hi + 1) >> 1;
        if ((int64_t)prefix2[mid] <= si) e = mid;
        else hi = mid - 1;
      }
      nt = u - si * n_tiles;
      mt = prefix[e + 1] - prefix[e];          // after the expert's full-cost tiles
    }
    const int s = slot ? slot[e] : e;
    int64_t lo = offsets[e];
    lo = lo < 0 ? 0 : (lo > max_rows ? max_rows : lo);
    int64_t hi = offsets[e + 1];
    hi = hi < lo ? lo : (hi > max_rows ? max_rows : hi);
    const int64_t row0 = lo + mt * BM;
    const int64_t row_end = min(row0 + (int64_t)BM, hi);
    const int64_t n0 = nt * kOutN;
    const int nrows = (int)(row_end - row0);

    // DMA sources: raw buffers over the tile's rows of A and of B (EPI 0: the
    // gate rows and the up rows apart), a 32-bit byte offset per lane and the
    // K offset as the scalar offset, so a K-step costs one scalar add. Rows
    // past the end of the expert or of the weight read the tile's first row;
    // their results are never stored.
    const int64_t rows_b = min((int64_t)kOutN, N_out - n0);
    const auto rs_a = make_rsrc(A + row0 * K, nrows * K);
    const auto rs_b0 = make_rsrc(B0 + ((int64_t)s * N_out + n0) * K, rows_b * K);
    const auto rs_b1 = make_rsrc((EPI == 0 ? B1 : B0) + ((int64_t)s * N_out + n0) * K, rows_b * K);
    uint32_t a_off[PPW], b_off[PPW];
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
      const int piece = wave * PPW + i;
      const int r = piece * ROWS_PER_PIECE + lrow;
      const int lch = swz(r, lpch);
      a_off[i] = (uint32_t)(((r < nrows ? r : 0) * K + lch * 8) * 2);
      // EPI 0: 32-row groups gate, up, gate, up, ... (two pieces each)
      const int wr = EPI == 0 ? (piece >> 2) * 32 + (r & 31) : r;
      b_off[i] = (uint32_t)(((wr < rows_b ? wr : 0) * K + lch * 8) * 2);
    }
    auto issue_a = [&](auto stage_c, int i, int64_t step) {
      constexpr int st = decltype(stage_c)::value;
      buf_dma16(rs_a, a_off[i], (uint32_t)((kbeg + step) * (BK * 2)), As[st] + (wave * PPW + i) * 512);
    };
    auto issue_b = [&](auto stage_c, int i, int64_t step) {
      constexpr int st = decltype(stage_c)::value;
      buf_dma16(i < PPW / 2 || EPI == 1 ? rs_b0 : rs_b1, b_off[i], (uint32_t)((kbeg + step) * (BK * 2)),
                Bs[st] + (wave * PPW + i) * 512);
    };
    // pieces [i0, i1) of the pair of steps (step, step + 1), both halves of a
    // line next to each other; steps past the end are left out
    auto pair_a = [&](auto st0, auto st1, int i0, int i1, int64_t step, int64_t nks) {
#pragma unroll
      for (int i = 0; i < PPW; ++i) {
        if (i < i0 || i >= i1) continue;
        if (step < nks) issue_a(st0, i, step);
        if (step + 1 < nks) issue_a(st1, i, step + 1);
      }
    };
    auto pair_b = [&](auto st0, auto st1, int64_t step, int64_t nks) {
#pragma unroll
      for (int i = 0; i < PPW; ++i) {
        if (step < nks) issue_b(st0, i, step);
        if (step + 1 < nks) issue_b(st1, i, step + 1);
      }
    };

    // MODE 0: 2 x 2 waves of 128 x 128; MODE m in {1, 2, 4}: 4 waves side by
    // side, each m x 32 rows by 64 columns.
    auto run = [&](auto mode_c) {
      constexpr int MODE = decltype(mode_c)::value;
      constexpr bool FULL = MODE == 0;
      constexpr int MI = FULL ? 8 : 2 * MODE;      // 16-row fragments
      constexpr int NI = FULL ? 8 : 4;             // 16-column fragments
      constexpr int MH = MI / 2;
      const int rbase = FULL ? (wave >> 1) * 128 : 0;
      const int cbase = FULL ? (wave & 1) * 128 : wave * 64;

      f32x4_t acc[MI][NI];
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          acc[mi][ni] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          asm volatile("" : "+a"(acc[mi][ni]));
        }
      asm volatile("s_nop 7");                     // register writes before the first MFMA
      // fragments of a K-step: the lower and upper halves of the A rows, and
      // the B columns of an even and an odd step
      bf16x8_t fal[MH], fah[MH], fb0[NI], fb1[NI];

      // Half a K-step: the MFMAs of one half of the A rows, in order, with the
      // fragment reads after its first MFMAs (one each) and four DMA pieces
      // spread over all of them; the fences keep this order.
      auto half_step = [&](int half, const bf16x8_t (&fa)[MH], const bf16x8_t (&fb)[NI], int n_rd,
                           auto&& read, auto&& dma) {
        constexpr int NM = MH * NI;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          mfma_acc(acc[half * MH + m / NI][m % NI], fa[m / NI], fb[m % NI]);
#pragma unroll
          for (int j = 0; j < MH + NI; ++j)
            if (j < n_rd && min(j, NM - 1) == m) read(j);
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if ((2 * k + 1) * NM / 8 == m) dma(k);
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      auto read_a1 = [&](auto stage_c, int half, int mi, bf16x8_t (&f)[MH]) {
        const int r = rbase + (half * MH + mi) * 16 + frow;
        f[mi] = *reinterpret_cast<const bf16x8_t*>(&As[decltype(stage_c)::value][r * BK + swz(r, fk) * 8]);
      };
      auto read_b1 = [&](auto stage_c, int ni, bf16x8_t (&f)[NI]) {
        const int r = cbase + ni * 16 + frow;
        f[ni] = *reinterpret_cast<const bf16x8_t*>(&Bs[decltype(stage_c)::value][r * BK + swz(r, fk) * 8]);
      };
      // the next step's fragments in the order its MFMAs take them
      auto read_next = [&](auto stage_c, int j, bf16x8_t (&fbn)[NI]) {
        if (j == 0) read_a1(stage_c, 0, 0, fal);
        else if (j <= NI) read_b1(stage_c, j - 1, fbn);
        else read_a1(stage_c, 0, j - NI, fal);
      };
      // K-steps run in pairs (e, e + 1), e even, over stages J = e mod 5 and
      // J + 1. After the barrier of the even step stage J has been read by
      // every wave, so the pair e + 4 can start to load into J + 4 and J; its
      // last A pieces go out in the next pair's first half-step. The wait in
      // the odd step is for the pair e + 2: younger are the eight B loads of
      // the pair e + 4.
      auto pair_ss = [&](auto j_c, int64_t kt) {
        constexpr int J = decltype(j_c)::value;
        using S0 = std::integral_constant<int, J>;
        using S1 = std::integral_constant<int, (J + 1) % 5>;
        using S2 = std::integral_constant<int, (J + 2) % 5>;
        using S3 = std::integral_constant<int, (J + 3) % 5>;
        using S4 = std::integral_constant<int, (J + 4) % 5>;
        half_step(0, fal, fb0, MH, [&](int j) { read_a1(S0{}, 1, j, fah); }, [&](int k) {
          if (k & 1) issue_a(S3{}, 2 + k / 2, kt + 3);
          else issue_a(S2{}, 2 + k / 2, kt + 2);
        });
        lds_barrier();
        half_step(1, fah, fb0, MH + NI, [&](int j) { read_next(S1{}, j, fb1); }, [&](int k) {
          if (k & 1) issue_b(S0{}, k / 2, kt + 5);
          else issue_b(S4{}, k / 2, kt + 4);
        });
        half_step(0, fal, fb1, MH, [&](int j) { read_a1(S1{}, 1, j, fah); }, [&](int k) {
          if (k & 1) issue_b(S0{}, 2 + k / 2, kt + 5);
          else issue_b(S4{}, 2 + k / 2, kt + 4);
        });
        wait_vmcnt<2 * PPW>();
        lds_barrier();
        half_step(1, fah, fb1, MH + NI, [&](int j) { read_next(S2{}, j, fb0); }, [&](int k) {
          if (k & 1) issue_a(S0{}, k / 2, kt + 5);
          else issue_a(S4{}, k / 2, kt + 4);
        });
      };
      // the same near the end of K: loads and reads past the end left out
      auto read_all = [&](auto stage_c, bf16x8_t (&fbn)[NI]) {
#pragma unroll
        for (int j = 0; j < MH + NI; ++j) read_next(stage_c, j, fbn);
      };
      auto pair_gen = [&](auto j_c, int64_t kt) {
        constexpr int J = decltype(j_c)::value;
        using S0 = std::integral_constant<int, J>;
        using S1 = std::integral_constant<int, (J + 1) % 5>;
        using S2 = std::integral_constant<int, (J + 2) % 5>;
        using S3 = std::integral_constant<int, (J + 3) % 5>;
        using S4 = std::integral_constant<int, (J + 4) % 5>;
        auto none = [](int) {};
        pair_a(S2{}, S3{}, 2, PPW, kt + 2, nks);
        half_step(0, fal, fb0, MH, [&](int j) { read_a1(S0{}, 1, j, fah); }, none);
        if (kt + 1 < nks) {
          lds_barrier();
          pair_b(S4{}, S0{}, kt + 4, nks);
          read_all(S1{}, fb1);
        }
        half_step(1, fah, fb0, 0, none, none);
        if (kt + 1 >= nks) return;
        half_step(0, fal, fb1, MH, [&](int j) { read_a1(S1{}, 1, j, fah); }, none);
        if (kt + 5 < nks) wait_vmcnt<2 * PPW>();
        else wait_vmcnt<0>();
        lds_barrier();
        pair_a(S4{}, S0{}, 0, PPW / 2, kt + 4, nks);
        if (kt + 2 < nks) read_all(S2{}, fb0);
        half_step(1, fah, fb1, 0, none, none);
      };

      pair_b(I0{}, I1{}, 0, nks);
      pair_a(I0{}, I1{}, 0, PPW, 0, nks);
      pair_b(I2{}, I3{}, 2, nks);
      pair_a(I2{}, I3{}, 0, PPW / 2, 2, nks);
      // the first pair has landed (LDS-only barrier: the second keeps loading)
      if (nks >= 4) wait_vmcnt<3 * PPW>();
      else wait_vmcnt<0>();
      lds_barrier();
      read_all(I0{}, fb0);
      int64_t kt = 0;
      for (; kt + 14 <= nks; kt += 10) {
        pair_ss(I0{}, kt);
        pair_ss(I2{}, kt + 2);
        pair_ss(I4{}, kt + 4);
        pair_ss(I1{}, kt + 6);
        pair_ss(I3{}, kt + 8);
      }
      for (; kt < nks; kt += 10) {
        pair_gen(I0{}, kt);
        if (kt + 2 < nks) pair_gen(I2{}, kt + 2);
        if (kt + 4 < nks) pair_gen(I4{}, kt + 4);
        if (kt + 6 < nks) pair_gen(I1{}, kt + 6);
        if (kt + 8 < nks) pair_gen(I3{}, kt + 8);
      }
      // every wave is past its last fragment reads before the epilogue
      // rewrites the stages; the last MFMAs' results are written
      lds_barrier();
      asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) asm volatile("" : "+a"(acc[mi][ni]));

      // A K-piece stores its fp32 partial tile; the piece that arrives last
      // (a device-scope counter per tail tile, ordered by release and acquire
      // fences) adds all pieces in piece order, so the sum does not depend on
      // arrival order, and writes the output.
      if (split_tile) {
        constexpr int kF4 = fast::kPieceBytes / 16 / 256;       // float4 per thread
        static_assert(MI * NI <= kF4, "partial tile layout");
        const int64_t tile_slot = t - full;
        f32x4_t* const P = reinterpret_cast<f32x4_t*>(partial);
        f32x4_t* const mine = P + (tile_slot * split + piece) * (int64_t)kF4 * 256;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) mine[(mi * NI + ni) * 256 + tid] = acc[mi][ni];
        __threadfence();
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(&tail[1 + tile_slot], 1) == (int)split - 1;
        __syncthreads();
        if (!s_last) return;
        __threadfence();
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (int64_t pc = 0; pc < split; ++pc) {
          const f32x4_t* const src = P + (tile_slot * split + pc) * (int64_t)kF4 * 256;
#pragma unroll
          for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) acc[mi][ni] += src[(mi * NI + ni) * 256 + tid];
        }
      }

      // Epilogue, staged through LDS (the stages are free: every wave passed
      // the last K-step's barrier after its last fragment read). Each wave
      // writes its bf16 results into the tile, 32 rows per stage array, with
      // the 16-byte chunks of a row XOR-swizzled by (row mod 8); then the
      // block stores whole rows with 16-byte coalesced writes.
      // 16x16 C layout: column lane % 16, rows 4 * (lane / 16) + q.
      constexpr int NOUT = kOutN;                       // output columns of the tile
      // Stage array holding rows [32 b, 32 b + 32) of the tile (b compile-time).
      auto stage_of = [&](auto b_c) -> uint16_t* {
        constexpr int b = decltype(b_c)::value;
        if constexpr (b < 4) return As[b];
        else return Bs[b - 4];
      };
      auto off_in = [](int r, int c) {               // r: row within the 32-row block
        return r * NOUT + ((((c >> 3) ^ (r & 7)) << 3) | (c & 7));
      };
      // Lane coordinates are made opaque per tile so that the write addresses
      // derived from them are formed here, not hoisted out of the tile loop.
      int ccol = lane & 15;
      int crow = (lane >> 4) * 4;
      asm volatile("" : "+v"(ccol), "+v"(crow));
      // wave's rows: 32-row blocks (rbase / 32) + mi / 2
      auto write_rows = [&](auto b0_c) {
        constexpr int B0 = decltype(b0_c)::value;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
          uint16_t* const base = mi < 2 ? stage_of(std::integral_constant<int, B0>{})
                               : mi < 4 ? stage_of(std::integral_constant<int, B0 + 1>{})
                               : mi < 6 ? stage_of(std::integral_constant<int, (B0 + 2) % 8>{})
                                        : stage_of(std::integral_constant<int, (B0 + 3) % 8>{});
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int r = (mi & 1) * 16 + crow + q;
            if (EPI == 0) {
              // 32-column groups: two gate fragments, then the two up fragments
#pragma unroll
              for (int p = 0; p < NI / 4; ++p)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                  const float g = acc[mi][4 * p + hh][q];
                  const float u = acc[mi][4 * p + 2 + hh][q];
                  base[off_in(r, cbase / 2 + p * 32 + hh * 16 + ccol)] = f32_to_bf16(swiglu(g, u));
                }
            } else {
#pragma unroll
              for (int ni = 0; ni < NI; ++ni)
                base[off_in(r, cbase + ni * 16 + ccol)] = f32_to_bf16(acc[mi][ni][q]);
            }
          }
        }
      };
      if (FULL && (wave >> 1)) write_rows(std::integral_constant<int, 4>{});
      else write_rows(std::integral_constant<int, 0>{});
      __syncthreads();
      // Rows of the tile that hold results: all 256 in a full tile, MI * 32
      // when the waves sit side by side.
      constexpr int CPRO = NOUT / 8;                    // 16-byte chunks per output row
      const int rows_here = min(nrows, FULL ? BM : MI * 32);
      int64_t ld = ldc;
      asm volatile("" : "+s"(ld));
      int tid_o = tid;
      asm volatile("" : "+v"(tid_o));
      auto store_block = [&](auto b_c) {
        constexpr int b = decltype(b_c)::value;
        const uint16_t* const base = stage_of(b_c);
#pragma unroll
        for (int qd0 = 0; qd0 < 32 * CPRO; qd0 += fast::kThreads) {
          const unsigned qd = qd0 + tid_o;
          const int r = qd / CPRO, ch = qd % CPRO;
          if (b * 32 + r < rows_here && n0 + ch * 8 < N_out) {
            const uint4 v = *reinterpret_cast<const uint4*>(base + off_in(r, ch * 8));
            *reinterpret_cast<uint4*>(C + (row0 + b * 32 + r) * ld + n0 + ch * 8) = v;
          }
        }
      };
      store_block(std::integral_constant<int, 0>{});
      store_block(std::integral_constant<int, 1>{});
      store_block(std::integral_constant<int, 2>{});
      store_block(std::integral_constant<int, 3>{});
      if (FULL) {
        store_block(std::integral_constant<int, 4>{});
        store_block(std::integral_constant<int, 5>{});
        store_block(std::integral_constant<int, 6>{});
        store_block(std::integral_constant<int, 7>{});
      }
    };
    if (nrows > 128) run(std::integral_constant<int, 0>{});
    else if (nrows > 64) run(std::integral_constant<int, 4>{});
    else if (nrows > 32) run(std::integral_constant<int, 2>{});
    else run(std::integral_constant<int, 1>{});
  }
}

// ---------------------------------------------------------------- f32 path
// float32 on the matrix cores (v_mfma_f32_16x16x4_f32: float32 products and
// sums). A block owns 16 output columns (of gate and of up, or of down) of at
// most 64 rows of one expert; its four waves split K in 16-wide steps, dealt
// round robin, and their partial sums are added through LDS in wave order. A
// lane loads 16 bytes = 4 neighbouring k of its row, and the v-th of them feeds
// the step's v-th MFMA, whose four k are then 4 apart, the same for both
// operands. Such small launches are bound by latency: enough blocks (16
// columns), short K chains and several loads in flight, instead of one thread
// that walks the whole of K for each output. Both projections: 8 experts, 128
// rows, H 128, F 256 76 -> 10 us; 4 experts, 1024 rows, H 512, F 1024 5687 ->
// 58 us.
constexpr int kF32Rows = 64, kF32Waves = 4;

template <int EPI>
__global__ void __launch_bounds__(64 * kF32Waves)
ffn_f32_mfma(const float* __restrict__ A, int64_t K, const float* __restrict__ B0,
             const float* __restrict__ B1, int64_t N_out, const int32_t* __restrict__ offsets,
             const int32_t* __restrict__ slot, int E, int S, int64_t max_rows,
             float* __restrict__ C) {
  constexpr int NB = EPI == 0 ? 2 : 1, RT = kF32Rows / 16;
  __shared__ f32x4_t part[kF32Waves][RT][NB][kWave];
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  // the expert and row group of this block: every wave counts the groups of
  // the experts before each lane's, 64 experts at a time
  int e = -1;
  int64_t group = 0, seen = 0;
  for (int e0 = 0; e0 < E && e < 0; e0 += kWave) {
    const int q = e0 + lane;
    const int64_t m = q < E ? expert_rows(offsets, slot, q, S, max_rows, nullptr) : 0;
    const int mine = (int)((m + kF32Rows - 1) / kF32Rows);
    int run = mine;
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(run, o, kWave);
      if (lane >= o) run += y;
    }
    const uint64_t hit = ballot(seen + run > (int64_t)blockIdx.y && seen + run - mine <= (int64_t)blockIdx.y);
    if (hit) {
      const int l = __ffsll((unsigned long long)hit) - 1;
      e = e0 + l;
      group = (int64_t)blockIdx.y - (seen + __shfl(run, l, kWave) - __shfl(mine, l, kWave));
    }
    seen += __shfl(run, kWave - 1, kWave);
  }
  if (e < 0) return;                             // past the last group (whole block)
  int64_t lo;
  const int64_t rows = expert_rows(offsets, slot, e, S, max_rows, &lo);
  const int s = slot ? slot[e] : e;
  const int64_t row0 = lo + group * kF32Rows;
  const int m = (int)min(rows - group * kF32Rows, (int64_t)kF32Rows);
  const int64_t n0 = (int64_t)blockIdx.x * 16;
  const int r = lane & 15, q = lane >> 4;
  // rows past m and columns past N_out read a valid row; not stored
  const float* a_row[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) a_row[i] = A + (row0 + min(16 * i + r, m - 1)) * K;
  const int64_t col = min(n0 + r, N_out - 1);
  const float* const b0 = B0 + ((int64_t)s * N_out + col) * K;
  const float* const b1 = EPI == 0 ? B1 + ((int64_t)s * N_out + col) * K : b0;
  const int rt = (m + 15) / 16;
  f32x4_t acc[RT][NB];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[i][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  for (int64_t k0 = wave * 16; k0 < K; k0 += 16 * kF32Waves) {
    const int64_t kk = k0 + 4 * q;               // K is a multiple of 4
    const bool in = kk < K;
    f32x4_t w[NB], a[RT];
    w[0] = in ? *reinterpret_cast<const f32x4_t*>(b0 + kk) : zero;
    if constexpr (EPI == 0) w[1] = in ? *reinterpret_cast<const f32x4_t*>(b1 + kk) : zero;
#pragma unroll
    for (int i = 0; i < RT; ++i)
      a[i] = in && i < rt ? *reinterpret_cast<const f32x4_t*>(a_row[i] + kk) : zero;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      if (i >= rt) continue;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][v], w[b][v], acc[i][b], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int b = 0; b < NB; ++b) part[wave][i][b][lane] = acc[i][b];
  __syncthreads();
  // wave i finishes row tile i; lane: column lane % 16, rows 4 * (lane / 16) + q
  static_assert(RT == kF32Waves, "one row tile per wave");
  if (wave >= rt || n0 + r >= N_out) return;
  f32x4_t t[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    t[b] = part[0][wave][b][lane];
#pragma unroll
    for (int w = 1; w < kF32Waves; ++w) t[b] += part[w][wave][b][lane];
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int rr = 16 * wave + 4 * q + v;
    if (rr >= m) continue;
    const float g = t[0][v];
    C[(row0 + rr) * N_out + n0 + r] = EPI == 0 ? g / (1.f + expf(-g)) * t[NB - 1][v] : g;
  }
}

__device__ __forceinline__ int expert_of_row(const int32_t* offsets, int E, int64_t r) {
  // last e with offsets[e] <= r (offsets non-decreasing)
  int lo = 0, hi = E;  // answer in [0, E)
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (offsets[mid] <= r) lo = mid; else hi = mid;
  }
  return lo;
}

__global__ void ffn_f32_up(const float* __restrict__ x, int64_t H, int64_t F,
                           const int32_t* __restrict__ offsets, const int32_t* __restrict__ slot,
                           int E, int S, int64_t max_rows, const float* __restrict__ wg,
                           const float* __restrict__ wu, float* __restrict__ act) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t r = q / F, f = q % F;
  if (r >= max_rows) return;
  const int64_t end = min((int64_t)offsets[E], max_rows);
  if (r < offsets[0] || r >= end) return;
  const int e = expert_of_row(offsets, E, r);
  const int s = slot ? slot[e] : e;
  if (s < 0 || s >= S) return;
  const float* xr = x + r * H;
  const float* g = wg + ((int64_t)s * F + f) * H;
  const float* u = wu + ((int64_t)s * F + f) * H;
  float sg = 0.f, su = 0.f;
  for (int64_t h = 0; h < H; ++h) {
    sg = fmaf(xr[h], g[h], sg);
    su = fmaf(xr[h], u[h], su);
  }
  act[r * F + f] = sg / (1.f + expf(-sg)) * su;
}

__global__ void ffn_f32_down(const float* __restrict__ act, int64_t H, int64_t F,
                             const int32_t* __restrict__ offsets, const int32_t* __restrict__ slot,
                             int E, int S, int64_t max_rows, const float* __restrict__ wd,
                             float* __restrict__ y) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t r = q / H, h = q % H;
  if (r >= max_rows) return;
  const int64_t end = min((int64_t)offsets[E], max_rows);
  if (r < offsets[0] || r >= end) return;
  const int e = expert_of_row(offsets, E, r);
  const int s = slot ? slot[e] : e;
  if (s < 0 || s >= S) return;
  const float* ar = act + r * F;
  const float* d = wd + ((int64_t)s * H + h) * F;
  float acc = 0.f;
  for (int64_t f = 0; f < F; ++f) acc = fmaf(ar[f], d[f], acc);
  y[r * H + h] = acc;
}

}  // namespace
}  // namespace moe

extern "C" size_t moe_expert_ffn_workspace(int64_t max_rows, int64_t H, int64_t F, int32_t E,
                                           int32_t dtype) {
  using namespace moe;
  if (max_rows < 1 || H < 1 || F < 1 || E < 1 || !valid_dtype(dtype)) return 0;
  const size_t elt = dtype == MOE_BF16 ? 2 : 4;
  size_t bytes = align_up((size_t)max_rows * (size_t)F * elt, 256);
  bytes += align_up((size_t)(E + 1 + kCounterWords + 2 * (E + 1)) * sizeof(int32_t), 256);
  if (dtype == MOE_BF16 && fast_path(H, F))
    bytes += (size_t)max_split_pieces(max_rows, H, F, E) * fast::kPieceBytes;
  return bytes;
}

extern "C" int moe_expert_ffn(const void* x_perm, int32_t dtype, int64_t max_rows, int64_t H,
                              int64_t F, const int32_t* expert_offsets, int32_t E,
                              const int32_t* slot_of_expert, int32_t S, const void* w_gate,
                              const void* w_up, const void* w_down, void* y_perm,
                              void* workspace, size_t ws_bytes, void* stream) {
  using namespace moe;
  MOE_CHECK_ARG(x_perm && expert_offsets && y_perm);
  MOE_CHECK_ARG(valid_dtype(dtype));
  MOE_CHECK_ARG(max_rows >= 1 && H >= 1 && F >= 1 && E >= 1 && E <= 256 && S >= 0);
  MOE_CHECK_ARG(slot_of_expert != nullptr || S >= E);
  MOE_CHECK_ARG(S == 0 || (w_gate && w_up && w_down));
  MOE_CHECK_ARG(max_rows < ((int64_t)1 << 31));
  if (dtype == MOE_BF16 && (H % 8 != 0 || F % 8 != 0)) return MOE_ERR_UNSUPPORTED;
  const size_t need = moe_expert_ffn_workspace(max_rows, H, F, E, dtype);
  if (!workspace || ws_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255))
    return MOE_ERR_WORKSPACE;
  if (S == 0) return MOE_OK;  // nothing resident: every row is a miss
  hipStream_t st = as_stream(stream);
  const size_t elt = dtype == MOE_BF16 ? 2 : 4;
  char* ws = static_cast<char*>(workspace);
  void* act = ws;
  int32_t* prefix = reinterpret_cast<int32_t*>(ws + align_up((size_t)max_rows * F * elt, 256));

  const uintptr_t at = reinterpret_cast<uintptr_t>(x_perm) | reinterpret_cast<uintptr_t>(w_gate) |
                       reinterpret_cast<uintptr_t>(w_up) | reinterpret_cast<uintptr_t>(w_down);
  if (dtype == MOE_F32) {
    // 16-byte loads, and a grid that covers every expert's row groups
    const int64_t groups = ceil_div(max_rows, kF32Rows) + std::min<int64_t>(E, max_rows);
    if (H % 4 == 0 && F % 4 == 0 && (at & 15) == 0 && groups <= 65535) {
      ffn_f32_mfma<0><<<dim3((unsigned)ceil_div(F, 16), (unsigned)groups), dim3(64 * kF32Waves), 0, st>>>(
          static_cast<const float*>(x_perm), H, static_cast<const float*>(w_gate),
          static_cast<const float*>(w_up), F, expert_offsets, slot_of_expert, E, S, max_rows,
          static_cast<float*>(act));
      MOE_CHECK_LAUNCH();
      ffn_f32_mfma<1><<<dim3((unsigned)ceil_div(H, 16), (unsigned)groups), dim3(64 * kF32Waves), 0, st>>>(
          static_cast<const float*>(act), F, static_cast<const float*>(w_down), nullptr, H,
          expert_offsets, slot_of_expert, E, S, max_rows, static_cast<float*>(y_perm));
      MOE_CHECK_LAUNCH();
      return MOE_OK;
    }
    const int64_t n1 = max_rows * F, n2 = max_rows * H;
    if (ceil_div(n1, 256) > 0x7fffffff || ceil_div(n2, 256) > 0x7fffffff) return MOE_ERR_UNSUPPORTED;
    ffn_f32_up<<<dim3((unsigned)ceil_div(n1, 256)), dim3(256), 0, st>>>(
        static_cast<const float*>(x_perm), H, F, expert_offsets, slot_of_expert, E, S, max_rows,
        static_cast<const float*>(w_gate), static_cast<const float*>(w_up), static_cast<float*>(act));
    MOE_CHECK_LAUNCH();
    ffn_f32_down<<<dim3((unsigned)ceil_div(n2, 256)), dim3(256), 0, st>>>(
        static_cast<const float*>(act), H, F, expert_offsets, slot_of_expert, E, S, max_rows,
        static_cast<const float*>(w_down), static_cast<float*>(y_perm));
    MOE_CHECK_LAUNCH();
    return MOE_OK;
  }

  // buffer loads and DMA of 16 bytes; the general path's loads take any address
  const bool fast = fast_path(H, F) && (at & 15) == 0;
  const int bm = fast ? fast::BM : BM;
  // Experts with at most 16 * kSmallMaxTiles rows go to the weight-streaming
  // kernel when the batch is decode-sized (at most 64 rows per expert on
  // average): bf16, H and F multiples of 32 (the fast-path shapes), 32-bit lane
  // offsets within 96 rows of K. Larger batches leave the rare small expert to
  // the large tiles and launch no few-row kernel at all.
  const bool few = fast && max_rows <= 64 * (int64_t)E;
  const int small_tiles = few ? kSmallMaxTiles : 0;
  // Whether an expert can hold more rows than one item decides if the large
  // tiles are launched beside it. They cost the tile list and two launches
  // that mostly find nothing (some 13 us); splitting such an expert into items
  // costs reading its weights once more per item, some 9 us for 54 MB. At
  // that size and below the few-row kernel takes every expert.
  const int64_t extra = few ? (max_rows - 1) / kSmallRows : 0;
  const bool only_few = few && extra * 6 * H * F <= 54 * 1000 * 1000;
  const bool big = !only_few;
  if (big) {
    ffn_tiles_kernel<<<dim3(1), dim3(kMaxExperts), 0, st>>>(expert_offsets, slot_of_expert, E, S,
                                                            max_rows, bm, small_tiles,
                                                            fast ? 1 : 0, prefix);
    MOE_CHECK_LAUNCH();
  }
  // without the large tiles the list (at most kMaxItems + 1 words) takes the
  // place of their prefix and counters
  int32_t* const small = only_few ? prefix : prefix + E + 1 + kCounterWords;
  static_assert(kMaxItems + 1 <= kCounterWords, "the item list fits the counters' words");
  const int32_t* const prefix2 = prefix + E + 1 + kCounterWords + E + 1;
  // the most row tiles an item can have, rounded up to a compiled bound
  const int64_t few_tiles = std::min<int64_t>(ceil_div(max_rows, 16), kSmallMaxTiles);
  const int mtmax = few_tiles <= 1 ? 1 : few_tiles <= 2 ? 2 : few_tiles <= 4 ? 4 : 6;
  int grid = device_cu_count();
  grid = std::min((grid + 7) / 8 * 8, kMaxTailTiles);     // a tail round has < grid tiles
  const auto* xb = static_cast<const uint16_t*>(x_perm);
  auto* ab = static_cast<uint16_t*>(act);
  const auto* wgb = static_cast<const uint16_t*>(w_gate);
  const auto* wub = static_cast<const uint16_t*>(w_up);
  const auto* wdb = static_cast<const uint16_t*>(w_down);
  auto* yb = static_cast<uint16_t*>(y_perm);
  if (fast) {
    int32_t* const claim = prefix + E + 1;
    int32_t* const tail = claim + kClaimWords;
    float* const partial = reinterpret_cast<float*>(
        reinterpret_cast<char*>(prefix) + align_up((size_t)(E + 1 + kCounterWords + 2 * (E + 1)) * 4, 256));
    const int pieces = (int)max_split_pieces(max_rows, H, F, E);
    // The few-row units: at most min(E, max_rows) + extra items. Two wide blocks
    // or one of the other shapes' per compute unit stride over them (more blocks
    // in flight spread the reads over more DRAM rows at once: 60 experts of 4
    // rows, H 2048, F 1408, 172 us, 184 with three; of 48 rows 258, 287; fewer
    // leave bandwidth unused).
    const int64_t items = std::min<int64_t>(E, max_rows) + extra;
    const int64_t cus = device_cu_count();
    auto launch_mt = [&](auto epi_c, auto shape_c, auto mt_c, const uint16_t* a, int64_t K,
                         const uint16_t* b0, const uint16_t* b1, uint16_t* c) {
      constexpr int EPI = decltype(epi_c)::value, SHAPE = decltype(shape_c)::value;
      using SS = SmallShape<EPI, SHAPE>;
      const int64_t units = items * ceil_div(EPI == 0 ? F : H, SS::COLS);
      const unsigned g = (unsigned)std::min<int64_t>((SHAPE == kWide ? 2 : 1) * cus, units);
      ffn_small_bf16<EPI, decltype(mt_c)::value, SHAPE><<<dim3(g), dim3(64 * SS::WAVES), 0, st>>>(
          a, K, b0, b1, F, H, expert_offsets, slot_of_expert, E, S, max_rows, only_few ? 1 : 0,
          small, c);
    };
    auto launch_mid = [&](auto epi_c, const uint16_t* a, int64_t K, const uint16_t* b0,
                          const uint16_t* b1, uint16_t* c) {
      const std::integral_constant<int, kMid> mid{};
      if (mtmax == 1) launch_mt(epi_c, mid, std::integral_constant<int, 1>{}, a, K, b0, b1, c);
      else launch_mt(epi_c, mid, std::integral_constant<int, 2>{}, a, K, b0, b1, c);
    };
    auto launch_shape = [&](auto epi_c, auto shape_c, const uint16_t* a, int64_t K,
                            const uint16_t* b0, const uint16_t* b1, uint16_t* c) {
      if (mtmax == 1) launch_mt(epi_c, shape_c, std::integral_constant<int, 1>{}, a, K, b0, b1, c);
      else if (mtmax == 2) launch_mt(epi_c, shape_c, std::integral_constant<int, 2>{}, a, K, b0, b1, c);
      else if (mtmax == 4) launch_mt(epi_c, shape_c, std::integral_constant<int, 4>{}, a, K, b0, b1, c);
      else launch_mt(epi_c, shape_c, std::integral_constant<int, 6>{}, a, K, b0, b1, c);
    };
    auto launch_small = [&](auto epi_c, const uint16_t* a, int64_t K, const uint16_t* b0,
                            const uint16_t* b1, uint16_t* c) {
      constexpr int EPI = decltype(epi_c)::value;
      const int64_t n_out = EPI == 0 ? F : H;
      if (items * ceil_div(n_out, SmallShape<EPI, kNarrow>::COLS) <= cus)
        launch_shape(epi_c, std::integral_constant<int, kNarrow>{}, a, K, b0, b1, c);
      else if (mtmax <= 2 && items * ceil_div(n_out, SmallShape<EPI, kMid>::COLS) <= cus)
        launch_mid(epi_c, a, K, b0, b1, c);
      else
        launch_shape(epi_c, std::integral_constant<int, kWide>{}, a, K, b0, b1, c);
    };
    if (big) {
      ffn_gemm_bf16_fast<0><<<dim3(grid), dim3(fast::kThreads), 0, st>>>(
          xb, H, wgb, wub, F, H, expert_offsets, slot_of_expert, E, max_rows, prefix,
          prefix2, claim, tail, partial, pieces, ab);
      MOE_CHECK_LAUNCH();
    }
    if (few) {
      launch_small(std::integral_constant<int, 0>{}, xb, H, wgb, wub, ab);
      MOE_CHECK_LAUNCH();
    }
    if (big) {
      ffn_gemm_bf16_fast<1><<<dim3(grid), dim3(fast::kThreads), 0, st>>>(
          ab, F, wdb, nullptr, F, H, expert_offsets, slot_of_expert, E, max_rows, prefix,
          prefix2, claim + 8, tail + kTailWords, partial, pieces, yb);
      MOE_CHECK_LAUNCH();
    }
    if (few) {
      launch_small(std::integral_constant<int, 1>{}, ab, F, wdb, nullptr, yb);
      MOE_CHECK_LAUNCH();
    }
    return MOE_OK;
  }
  ffn_gemm_bf16<0><<<dim3(grid), dim3(kThreads), 0, st>>>(
      xb, H, wgb, wub, F, H, expert_offsets, slot_of_expert, E, max_rows, prefix, ab);
  MOE_CHECK_LAUNCH();
  ffn_gemm_bf16<1><<<dim3(grid), dim3(kThreads), 0, st>>>(
      ab, F, wdb, nullptr, F, H, expert_offsets, slot_of_expert, E, max_rows, prefix, yb);
  MOE_CHECK_LAUNCH();
  return MOE_OK;
}
