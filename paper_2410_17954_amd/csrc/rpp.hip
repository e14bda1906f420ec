// Forward pass of the routing path predictor (Sec. 3.2): a T5-style
// encoder-decoder whose L heads give every token logits over the E experts of
// each MoE layer, and their sigmoids as activation probabilities (B, S, L, E).
// Everything is float32. Hidden size 32 (the paper's) runs on float32 MFMAs,
// with everything between two attentions in one kernel per block of rows
// (rpp_rows32) and, for heads of 8, attention on MFMAs too (rpp_attention8);
// other sizes run as LDS-tiled vector kernels, one per step.
#include "moeflow.h"
#include "common.h"

#include <algorithm>
#include <vector>

namespace moe {
namespace {

constexpr int kMaxThr = 32;

// Relative-position buckets of one stack (T5): distance n = query - key.
struct RelBuckets {
  int bidirectional;
  int side;        // buckets per sign (num_buckets, or half of it when bidirectional)
  int m;           // exact buckets: distances 0 .. m-1
  int D;           // max_distance: n >= D falls in the last bucket
  int nthr;        // bucket of m <= n < D is m + (number of thr[] <= n)
  int thr[kMaxThr];
};

__device__ __forceinline__ int rel_bucket(const RelBuckets& rb, int n) {
  int ret = 0;
  if (rb.bidirectional) {
    if (n < 0) {
      ret = rb.side;
      n = -n;
    }
  } else if (n < 0) {
    n = 0;
  }
  if (n < rb.m) return ret + n;
  if (n >= rb.D) return ret + rb.side - 1;
  int j = 0;
  for (int q = 0; q < rb.nthr; ++q) j += rb.thr[q] <= n;
  return ret + min(rb.m + j, rb.side - 1);
}

// floor(log2(x)) of a positive 128-bit integer
int ilog2_u128(unsigned __int128 x) {
  int r = -1;
  while (x) {
    x >>= 1;
    ++r;
  }
  return r;
}

// Host: the exact logarithmic buckets. With m and D powers of two the bucket
// of m <= n < D is m + floor((floor(log2(n^a)) - a*log2(m)) / c), a = side - m,
// c = log2(D/m); thr[j-1] = the smallest n with bucket >= m + j.
bool make_buckets(bool bidirectional, int num_buckets, int max_distance, RelBuckets* rb) {
  rb->bidirectional = bidirectional ? 1 : 0;
  rb->side = bidirectional ? num_buckets / 2 : num_buckets;
  rb->m = rb->side / 2;
  rb->D = max_distance;
  const int m = rb->m, a = rb->side - m;
  auto pow2 = [](int v) { return v > 0 && (v & (v - 1)) == 0; };
  if (m < 1 || !pow2(m) || !pow2(max_distance) || max_distance <= m || a > 16) return false;
  const int lm = ilog2_u128(m), c = ilog2_u128((unsigned __int128)(max_distance / m));
  rb->nthr = 0;
  int prev = m;
  for (int n = m; n < max_distance; ++n) {
    unsigned __int128 p = 1;
    for (int q = 0; q < a; ++q) p *= (unsigned __int128)n;   // n < D <= 2^7 keeps n^16 < 2^112
    const int b = std::min(m + (ilog2_u128(p) - a * lm) / c, rb->side - 1);
    while (prev < b) {
      if (rb->nthr >= kMaxThr) return false;
      rb->thr[rb->nthr++] = n;
      ++prev;
    }
  }
  return true;
}

__global__ void rpp_embed(const int32_t* __restrict__ ids, int64_t M, int V, int d,
                          const float* __restrict__ emb, float* __restrict__ x,
                          int32_t* __restrict__ err) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q >= M * d) return;
  const int64_t t = q / d;
  const int c = (int)(q - t * d);
  const int id = ids[t];
  if (id < 0 || id >= V) {
    if (c == 0) atomicExch(err, 1);
    x[q] = 0.f;
    return;
  }
  x[q] = emb[(int64_t)id * d + c];
}

// out = x / sqrt(mean(x^2) + eps) * w; 32 lanes per row (lane c takes columns
// c, c + 32, ...), the sum of squares reduced across them in a fixed order.
__global__ void __launch_bounds__(256)
rpp_rmsnorm(const float* __restrict__ x, int64_t M, int d, const float* __restrict__ w,
            float eps, float* __restrict__ out) {
  const int64_t t = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 5;
  const int lane = threadIdx.x & 31;
  const bool live = t < M;
  const float* r = x + (live ? t : 0) * d;
  float ss = 0.f;
  if (live)
    for (int c = lane; c < d; c += 32) ss += r[c] * r[c];
  for (int o = 16; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 32);
  if (!live) return;
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int c = lane; c < d; c += 32) out[t * d + c] = r[c] * inv * w[c];
}

enum GemmMode { G_STORE = 0, G_ADD = 1, G_RELU = 2, G_SIGMOID = 3 };

// C[M, N] (op)= A[M, K] . W[N, K]^T. 256 threads as 16 x 16, each TM x TN
// outputs (rows ty + 16 i, columns tx + 16 j); K in steps of 16 through LDS.
// G_SIGMOID stores the logits to C and their sigmoids to P.
template <int TM, int TN, int MODE>
__global__ void __launch_bounds__(256)
rpp_gemm(const float* __restrict__ A, int64_t lda, const float* __restrict__ W, int64_t M,
         int64_t N, int64_t K, float* __restrict__ C, int64_t ldc, float* __restrict__ P) {
  constexpr int BM = 16 * TM, BN = 16 * TN, BK = 16;
  __shared__ float As[BK][BM + 1];
  __shared__ float Ws[BK][BN + 1];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = (int64_t)blockIdx.x * BN;
  float acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = 0.f;
  for (int64_t k0 = 0; k0 < K; k0 += BK) {
    for (int q = threadIdx.x; q < BM * BK; q += 256) {
      const int r = q / BK, c = q % BK;
      const int64_t gr = m0 + r, gc = k0 + c;
      As[c][r] = (gr < M && gc < K) ? A[gr * lda + gc] : 0.f;
    }
    for (int q = threadIdx.x; q < BN * BK; q += 256) {
      const int r = q / BK, c = q % BK;
      const int64_t gr = n0 + r, gc = k0 + c;
      Ws[c][r] = (gr < N && gc < K) ? W[gr * K + gc] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[kk][ty + 16 * i];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = Ws[kk][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t r = m0 + ty + 16 * i;
    if (r >= M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int64_t c = n0 + tx + 16 * j;
      if (c >= N) continue;
      float v = acc[i][j];
      if (MODE == G_ADD) v += C[r * ldc + c];
      if (MODE == G_RELU) v = fmaxf(v, 0.f);
      C[r * ldc + c] = v;
      if (MODE == G_SIGMOID) P[r * ldc + c] = 1.0f / (1.0f + __expf(-v));
    }
  }
}

// Attention of (sequence b, head h) for 64 queries per block: softmax over
// keys j of q_i . k_j (+ the bias of distance i - j) with j <= i when causal,
// then the weighted sum of v_j. Keys, values and the head's bias per distance
// (2S - 1 values) are staged in LDS; each query's keys are split over kSplit
// neighbouring lanes (key j goes to lane j mod kSplit), whose running softmax
// states are merged with lane shuffles in a fixed order.
constexpr int kAttQ = 64, kSplit = 4;
template <int DK>
__global__ void __launch_bounds__(kAttQ * kSplit)
rpp_attention(const float* __restrict__ Q, int64_t ldq, const float* __restrict__ Kp,
              const float* __restrict__ Vp, int64_t ldkv, int S, int h_count,
              const float* __restrict__ rel, RelBuckets rb, int use_bias, int causal,
              float* __restrict__ O, int64_t ldo) {
  extern __shared__ float kv_lds[];
  float* const ks = kv_lds;
  float* const vs = kv_lds + (size_t)S * DK;
  float* const bt = vs + (size_t)S * DK;              // bias of distance n at bt[n + S - 1]
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t base = (int64_t)b * S;
  for (int q = threadIdx.x; q < S * DK; q += blockDim.x) {
    const int j = q / DK, c = q % DK;
    ks[q] = Kp[(base + j) * ldkv + h * DK + c];
    vs[q] = Vp[(base + j) * ldkv + h * DK + c];
  }
  if (use_bias)
    for (int q = threadIdx.x; q < 2 * S - 1; q += blockDim.x)
      bt[q] = rel[rel_bucket(rb, q - (S - 1)) * h_count + h];
  __syncthreads();
  const int split = threadIdx.x % kSplit;
  const int i = blockIdx.x * kAttQ + threadIdx.x / kSplit;
  const bool live = i < S;
  float qv[DK], acc[DK];
#pragma unroll
  for (int c = 0; c < DK; ++c) {
    qv[c] = live ? Q[(base + i) * ldq + h * DK + c] : 0.f;
    acc[c] = 0.f;
  }
  float mx = -INFINITY, den = 0.f;
  const int jend = !live ? 0 : (causal ? i + 1 : S);
  for (int j = split; j < jend; j += kSplit) {
    float sc = 0.f;
#pragma unroll
    for (int c = 0; c < DK; ++c) sc = fmaf(qv[c], ks[j * DK + c], sc);
    if (use_bias) sc += bt[i - j + S - 1];
    const float nm = fmaxf(mx, sc);
    const float scale = __expf(mx - nm), p = __expf(sc - nm);
    den = den * scale + p;
#pragma unroll
    for (int c = 0; c < DK; ++c) acc[c] = fmaf(p, vs[j * DK + c], acc[c] * scale);
    mx = nm;
  }
  // merge the kSplit states of a query (lanes 4q .. 4q+3): pairs at distance 1, then 2
#pragma unroll
  for (int o = 1; o < kSplit; o <<= 1) {
    const float m2 = __shfl_xor(mx, o), d2 = __shfl_xor(den, o);
    const float nm = fmaxf(mx, m2);
    const float s1 = mx == -INFINITY ? 0.f : __expf(mx - nm);
    const float s2 = m2 == -INFINITY ? 0.f : __expf(m2 - nm);
    den = den * s1 + d2 * s2;
#pragma unroll
    for (int c = 0; c < DK; ++c) {
      const float a2 = __shfl_xor(acc[c], o);
      acc[c] = acc[c] * s1 + a2 * s2;
    }
    mx = nm;
  }
  if (!live || split != 0) return;
  const float inv = 1.0f / den;
#pragma unroll
  for (int c = 0; c < DK; ++c) O[(base + i) * ldo + h * DK + c] = acc[c] * inv;
}

// The same for heads of 8 on float32 MFMAs (16x16x4). A wave owns 16 queries and
// walks the keys 64 at a time: scores^T = K . Q^T puts 4 x 4 keys of one query
// in each lane (query lane % 16, keys 16 t + 4 (lane / 16) + v), and that is the
// operand layout of O^T = V^T . P^T, so the probabilities go from one product
// into the next in registers. The running maximum is common to a query's four
// lanes (two shuffles per 64 keys), the sums are merged at the end. The vector
// form spent four 16-byte LDS reads and some thirty vector operations per
// (query, key) pair: 34.8 us at 16 x 512 tokens.
constexpr int kAtt8Threads = 512, kAtt8Q = kAtt8Threads / kWave * 16;   // queries per block
template <bool BIAS>
__global__ void __launch_bounds__(kAtt8Threads)
rpp_attention8(const float* __restrict__ Q, int64_t ldq, const float* __restrict__ Kp,
               const float* __restrict__ Vp, int64_t ldkv, int S, int h_count,
               const float* __restrict__ rel, RelBuckets rb, int causal, float* __restrict__ O,
               int64_t ldo) {
  constexpr int DK = 8;
  extern __shared__ __attribute__((aligned(16))) float att_lds[];
  const int S64 = (S + 63) / 64 * 64;
  const int vp = S64 + 4;                            // pitch of a V^T row
  float* const ks = att_lds;                         // [S64][8]
  float* const vt = ks + (size_t)S64 * DK;           // [8][vp]
  float* const bt = vt + (size_t)DK * vp;            // bias of distance n at bt[n + S - 1]
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t base = (int64_t)b * S;
  // half rows of 16 bytes (row strides and head offsets are multiples of 4
  // floats); keys past the end: zeros, masked below
#pragma unroll 2
  for (int q = threadIdx.x; q < S64 * 2; q += kAtt8Threads) {
    const int j = q >> 1, c = (q & 1) * 4;
    float4 kk = make_float4(0.f, 0.f, 0.f, 0.f), vv = kk;
    if (j < S) {
      kk = *reinterpret_cast<const float4*>(Kp + (base + j) * ldkv + h * DK + c);
      vv = *reinterpret_cast<const float4*>(Vp + (base + j) * ldkv + h * DK + c);
    }
    *reinterpret_cast<float4*>(ks + j * DK + c) = kk;
    vt[c * vp + j] = vv.x;
    vt[(c + 1) * vp + j] = vv.y;
    vt[(c + 2) * vp + j] = vv.z;
    vt[(c + 3) * vp + j] = vv.w;
  }
  if (BIAS)
    for (int q = threadIdx.x; q < 2 * S - 1; q += kAtt8Threads)
      bt[q] = rel[rel_bucket(rb, q - (S - 1)) * h_count + h];
  __syncthreads();
  const int lane = lane_id();
  const int i0 = blockIdx.x * kAtt8Q + threadIdx.x / kWave * 16;
  if (i0 >= S) return;
  const int r = lane & 15, q4 = lane >> 4;
  const int i = min(i0 + r, S - 1);                  // queries past the end repeat the last
  const float* const qrow = Q + (base + i) * ldq + h * DK;
  const float q0 = qrow[2 * q4], q1 = qrow[2 * q4 + 1];
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};                // O^T: rows 0-7 are the head's columns
  float mx = -INFINITY, den = 0.f;
  const int jend = causal ? min(S, i0 + 16) : S;
  for (int j0 = 0; j0 < jend; j0 += 64) {
    f32x4_t sc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float2 kk = *reinterpret_cast<const float2*>(ks + (j0 + 16 * t + r) * DK + 2 * q4);
      sc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      sc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kk.x, q0, sc[t], 0, 0, 0);
      sc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kk.y, q1, sc[t], 0, 0, 0);
    }
    const bool edge = j0 + 64 > S || (causal && j0 + 63 > i0);   // wave-uniform
    float m = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = j0 + 16 * t + 4 * q4 + v;
        if (BIAS) sc[t][v] += bt[max(i - j, 1 - S) + S - 1];
        if (edge && (j >= S || (causal && j > i))) sc[t][v] = -INFINITY;
        m = fmaxf(m, sc[t][v]);
      }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    const float nm = fmaxf(mx, m);                   // finite: key 0 is never masked
    const float scale = __expf(mx - nm);
    mx = nm;
    den *= scale;
    // the block's own sum first: chains of 64 products, then one per 64 keys
    // (the causal diagonal: keys past the first query are masked for some of
    // the queries, p = 0, and a value of theirs that is not finite stays out of
    // the products)
    const bool diagonal = causal && j0 + 63 > i0;
    bool odd = false;
    f32x4_t blk = {0.f, 0.f, 0.f, 0.f};
    float dblk = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float4 vv = *reinterpret_cast<const float4*>(vt + (r & 7) * vp + j0 + 16 * t + 4 * q4);
      float va[4] = {vv.x, vv.y, vv.z, vv.w};
      if (diagonal)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j0 + 16 * t + 4 * q4 + v > i0 && !isfinite(va[v])) {
            va[v] = 0.f;
            odd = true;
          }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float p = __expf(sc[t][v] - nm);
        dblk += p;
        blk = __builtin_amdgcn_mfma_f32_16x16x4f32(va[v], p, blk, 0, 0, 0);
      }
    }
    den += dblk;
    if (ballot(odd)) {                               // for the queries that see them
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float p = __expf(sc[t][v] - nm);
          for (int g = 0; g < 4; ++g) {
            const int j = j0 + 16 * t + 4 * g + v;
            const float pj = __shfl(p, r + 16 * g);
            if (j <= i0 || j > i0 + r) continue;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float val = vt[((4 * q4 + c) & 7) * vp + j];
              if (!isfinite(val)) blk[c] = fmaf(pj, val, blk[c]);
            }
          }
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = fmaf(acc[v], scale, blk[v]);
  }
  den += __shfl_xor(den, 16);
  den += __shfl_xor(den, 32);
  if (q4 >= 2 || i0 + r >= S) return;                // O^T rows 4 q4 + v, columns queries
  const float inv = 1.0f / den;
  float* const o = O + (base + i) * ldo + h * DK + 4 * q4;
#pragma unroll
  for (int v = 0; v < 4; ++v) o[v] = acc[v] * inv;
}

// ---------------------------------------------------------- rows of width 32
// Everything a row of hidden size 32 goes through between two attentions, in
// one kernel over 16 * RT rows a block: the attention's output projection and
// residual, RMS norm, and either
//   kRowsCross  the cross-attention's query and its keys and values (from the
//               encoder output), or
//   kRowsMlp    the feed-forward block with its residual, the next RMS norm and
//               the next query/key/value projection (or, after a stack, the
//               normalised rows alone);
//   kRowsEmbed  starts a stack: embedding, norm, query/key/value.
// All products are float32 MFMAs (16x16x4) computed transposed, out^T = W .
// rows^T: a lane loads 16 bytes of a weight row and of a row of x (4
// neighbouring k, one for each of four MFMAs), and the result, 4 neighbouring
// outputs of one row per lane, is both a 16-byte store and the operand layout
// of the next product, so the feed-forward's hidden units stay in registers.
// Its width is dealt to the waves 16 units at a time, the partial sums are
// added in wave order. What bounds it: the MFMAs of the feed-forward (14 us of
// a 16 x 512 token batch at the float32 peak); as vector kernels, with the
// products around it in 11 launches per layer, the feed-forward alone took 104.
constexpr int kRowsEmbed = 0, kRowsCross = 1, kRowsMlp = 2;

struct Rows32 {
  int64_t M;
  float eps;
  const int32_t* ids;                  // embed
  const float* emb;
  int vocab;
  int32_t* err;
  float* x;                            // the residual stream [M, 32]
  const float* o;                      // attention output [M, 32]
  const float* wout;                   // its projection [32, 32]
  const float* ln;                     // the norm after it (embed: the only one)
  const float *w1, *w2;                // feed-forward [dff, 32], [32, dff]
  int dff;
  const float* ln_next;                // the norm after the feed-forward
  const float* wnext;                  // projection of the normalised rows [n_next, 32]
  int n_next;                          // 0: store the normalised rows
  float* next;                         // [M, n_next] or [M, 32]
  const float* enc;                    // cross: encoder output, wkv [64, 32] -> kv [M, 64]
  const float* wkv;
  float* kv;
};

template <int MODE, int RT, int NW>
__global__ void __launch_bounds__(64 * NW)
rpp_rows32(Rows32 a) {
  constexpr int R = 16 * RT, D = 32, P = D + 4;      // pitch: 16-byte rows, spread over banks
  __shared__ __attribute__((aligned(16))) float xs[R][P], ns[R][P];
  __shared__ __attribute__((aligned(16))) float part[MODE == kRowsMlp ? NW : 1][R][P];
  const int tid = threadIdx.x;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int c16 = lane & 15, q4 = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * R;
  auto row_at = [&](int r) { return min(r0 + r, a.M - 1); };   // rows past M repeat the last

  // B operand of 16 rows: lane (row c16, q4) holds k = 16 s + 4 q4 + v at [4 s + v]
  auto rows_of = [&](const float* p, float (&f)[8]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const float4 u = *reinterpret_cast<const float4*>(p + 16 * s + 4 * q4);
      f[4 * s] = u.x;
      f[4 * s + 1] = u.y;
      f[4 * s + 2] = u.z;
      f[4 * s + 3] = u.w;
    }
  };
  // 16 outputs (weight rows w, row stride D) of those 16 rows
  auto product = [&](const float* w, const float (&f)[8]) {
    float g[8];
    rows_of(w + (int64_t)c16 * D, g);
    f32x4_t d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 8; ++k) d = __builtin_amdgcn_mfma_f32_16x16x4f32(g[k], f[k], d, 0, 0, 0);
    return d;
  };
  // ns = rms(xs) * w, 64 NW / R threads a row
  auto norm = [&](const float* w) {
    constexpr int TPR = 64 * NW / R, PER = D / TPR;
    static_assert(TPR <= 32 && PER >= 1, "threads per row");
    const int r = tid / TPR, c = tid % TPR * PER;
    float v[PER], ss = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      v[j] = xs[r][c + j];
      ss += v[j] * v[j];
    }
#pragma unroll
    for (int o = TPR / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    const float inv = 1.0f / sqrtf(ss / (float)D + a.eps);
#pragma unroll
    for (int j = 0; j < PER; ++j) ns[r][c + j] = v[j] * inv * w[c + j];
  };
  // out[row, 0..n) = ns . w^T, the 16 x 16 tiles dealt to the waves
  auto project = [&](const float* w, int n, float* out) {
    const int tiles = (n / 16) * RT;
    for (int t = wave; t < tiles; t += NW) {
      const int rt = t % RT, ot = t / RT;
      float f[8];
      rows_of(&ns[16 * rt + c16][0], f);
      const f32x4_t d = product(w + (int64_t)ot * 16 * D, f);
      const int64_t row = r0 + 16 * rt + c16;
      if (row < a.M) *reinterpret_cast<f32x4_t*>(out + row * n + 16 * ot + 4 * q4) = d;
    }
  };

  if constexpr (MODE == kRowsEmbed) {
    for (int q = tid; q < R * D; q += 64 * NW) {
      const int r = q / D, c = q % D;
      const int id = a.ids[row_at(r)];
      const bool ok = id >= 0 && id < a.vocab;
      if (!ok && c == 0 && r0 + r < a.M) atomicExch(a.err, 1);
      const float v = ok ? a.emb[(int64_t)id * D + c] : 0.f;
      xs[r][c] = v;
      if (r0 + r < a.M) a.x[(r0 + r) * D + c] = v;
    }
    __syncthreads();
    norm(a.ln);
    __syncthreads();
    project(a.wnext, a.n_next, a.next);
    return;
  }

  for (int t = wave; t < 2 * RT; t += NW) {          // x += o . wout^T
    const int rt = t % RT, ot = t / RT;
    const int64_t row = row_at(16 * rt + c16);
    float f[8];
    rows_of(a.o + row * D, f);
    const float4 xo = *reinterpret_cast<const float4*>(a.x + row * D + 16 * ot + 4 * q4);
    const f32x4_t d = product(a.wout + (int64_t)ot * 16 * D, f);
    *reinterpret_cast<float4*>(&xs[16 * rt + c16][16 * ot + 4 * q4]) =
        make_float4(xo.x + d[0], xo.y + d[1], xo.z + d[2], xo.w + d[3]);
  }
  __syncthreads();
  norm(a.ln);
  __syncthreads();
  auto store_x = [&]() {
    for (int q = tid; q < R * D / 4; q += 64 * NW) {
      const int r = q / (D / 4), c = q % (D / 4) * 4;
      if (r0 + r < a.M)
        *reinterpret_cast<float4*>(a.x + (r0 + r) * D + c) = *reinterpret_cast<const float4*>(&xs[r][c]);
    }
  };
  if constexpr (MODE == kRowsCross) {
    store_x();
    project(a.wnext, a.n_next, a.next);
    for (int t = wave; t < 4 * RT; t += NW) {        // kv = enc . wkv^T
      const int rt = t % RT, ot = t / RT;
      const int64_t row = r0 + 16 * rt + c16;
      float f[8];
      rows_of(a.enc + row_at(16 * rt + c16) * D, f);
      const f32x4_t d = product(a.wkv + (int64_t)ot * 16 * D, f);
      if (row < a.M) *reinterpret_cast<f32x4_t*>(a.kv + row * 64 + 16 * ot + 4 * q4) = d;
    }
    return;
  }
  // feed-forward: hidden units 16 c .. 16 c + 15 of chunk c, chunks dealt to the
  // waves; the next chunk's weights load while this one's products run
  float f[RT][8];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) rows_of(&ns[16 * rt + c16][0], f[rt]);
  // sums in two levels, kSumChunks chunks (128 products) a chain: no longer
  // chains, so no larger rounding error, than the vector kernels' parts of 256
  constexpr int kSumChunks = 8;
  f32x4_t acc[RT][2], sum[RT][2];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ot = 0; ot < 2; ++ot) acc[rt][ot] = sum[rt][ot] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int chunks = (a.dff + 15) / 16;
  f32x4_t w1[2], w2[2];
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  auto fetch = [&](int c, f32x4_t (&u1)[2], f32x4_t (&u2)[2]) {
    const int h1 = 16 * c + c16, h2 = 16 * c + 4 * q4;         // dff is a multiple of 4
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      u1[s] = h1 < a.dff ? *reinterpret_cast<const f32x4_t*>(a.w1 + (int64_t)h1 * D + 16 * s + 4 * q4) : zero;
      u2[s] = h2 < a.dff ? *reinterpret_cast<const f32x4_t*>(a.w2 + (int64_t)(16 * s + c16) * a.dff + h2) : zero;
    }
  };
  if (wave < chunks) fetch(wave, w1, w2);
  int in_chain = 0;
  for (int c = wave; c < chunks; c += NW) {
    if (in_chain++ == kSumChunks) {
      in_chain = 1;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ot = 0; ot < 2; ++ot) {
          sum[rt][ot] += acc[rt][ot];
          acc[rt][ot] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
    f32x4_t n1[2] = {zero, zero}, n2[2] = {zero, zero};
    if (c + NW < chunks) fetch(c + NW, n1, n2);
    f32x4_t hid[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) hid[rt] = zero;
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        hid[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[k / 4][k % 4], f[rt][k], hid[rt], 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float hv = fmaxf(hid[rt][v], 0.f);
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
          acc[rt][ot] = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[ot][v], hv, acc[rt][ot], 0, 0, 0);
      }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      w1[s] = n1[s];
      w2[s] = n2[s];
    }
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ot = 0; ot < 2; ++ot)
      *reinterpret_cast<f32x4_t*>(&part[MODE == kRowsMlp ? wave : 0][16 * rt + c16][16 * ot + 4 * q4]) =
          sum[rt][ot] + acc[rt][ot];
  __syncthreads();
  for (int q = tid; q < R * D; q += 64 * NW) {
    const int r = q / D, c = q % D;
    float v = part[0][r][c];
#pragma unroll
    for (int w = 1; w < (MODE == kRowsMlp ? NW : 1); ++w) v += part[w][r][c];
    xs[r][c] += v;
  }
  __syncthreads();
  norm(a.ln_next);
  store_x();
  __syncthreads();
  if (a.n_next > 0) {
    project(a.wnext, a.n_next, a.next);
  } else {
    for (int q = tid; q < R * D; q += 64 * NW) {
      const int r = q / D, c = q % D;
      if (r0 + r < a.M) a.next[(r0 + r) * D + c] = ns[r][c];
    }
  }
}

constexpr int kMlpRows = 32, kMlpChunk = 64, kMlpSplit = 8;   // fused feed-forward tiles

struct RppOffsets {
  size_t emb, enc_rel, enc_ln, dec_rel, dec_ln, heads, total;
  std::vector<size_t> enc, dec;      // first value of each layer
};

size_t enc_layer_size(const moe_rpp_dims& g) {
  const size_t d = g.d_model, f = g.d_ff;
  return 2 * d + 4 * d * d + 2 * d * f;
}
size_t dec_layer_size(const moe_rpp_dims& g) {
  const size_t d = g.d_model, f = g.d_ff;
  return 3 * d + 8 * d * d + 2 * d * f;
}

RppOffsets rpp_offsets(const moe_rpp_dims& g) {
  RppOffsets o{};
  const size_t d = g.d_model;
  size_t p = 0;
  o.emb = p;
  p += (size_t)g.vocab * d;
  o.enc_rel = p;
  p += (size_t)g.num_buckets * g.n_heads;
  for (int l = 0; l < g.n_enc; ++l) {
    o.enc.push_back(p);
    p += enc_layer_size(g);
  }
  o.enc_ln = p;
  p += d;
  o.dec_rel = p;
  p += (size_t)g.num_buckets * g.n_heads;
  for (int l = 0; l < g.n_dec; ++l) {
    o.dec.push_back(p);
    p += dec_layer_size(g);
  }
  o.dec_ln = p;
  p += d;
  o.heads = p;
  p += (size_t)g.L * g.E * d;
  o.total = p;
  return o;
}

struct RppWs {
  size_t x, y, n, enc, o, qkv, kv, hid, logits, total;
};

RppWs rpp_ws(int64_t M, const moe_rpp_dims& g) {
  RppWs w{};
  size_t off = 0;
  auto take = [&](size_t floats) {
    const size_t at = off;
    off = align_up(off + floats * 4, 256);
    return at;
  };
  const size_t d = g.d_model;
  w.x = take(M * d);
  w.y = take(M * d);
  w.n = take(M * d);
  w.enc = take(M * d);
  w.o = take(M * d);
  w.qkv = take(M * 3 * d);
  w.kv = take(M * 2 * d);
  w.hid = take(M * (size_t)std::max(g.d_ff, kMlpSplit * g.d_model));
  w.logits = take(M * (size_t)g.L * g.E);
  w.total = off;
  return w;
}

bool dims_ok(const moe_rpp_dims* g) {
  if (!g) return false;
  return g->vocab >= 1 && g->d_model >= 1 && g->n_heads >= 1 && g->d_model % g->n_heads == 0 &&
         g->d_ff >= 1 && g->n_enc >= 0 && g->n_dec >= 0 && g->L >= 1 && g->E >= 1 &&
         g->num_buckets >= 2 && g->num_buckets % 2 == 0 && g->max_distance >= 1 && g->eps >= 0.f;
}

template <int MODE>
int gemm(hipStream_t st, const float* A, int64_t lda, const float* W, int64_t M, int64_t N,
         int64_t K, float* C, int64_t ldc, float* P = nullptr) {
  if (N <= 48) {                                  // narrow outputs: 32 x 32 tiles, more blocks
    const dim3 grid((unsigned)ceil_div(N, 32), (unsigned)ceil_div(M, 32));
    rpp_gemm<2, 2, MODE><<<grid, dim3(256), 0, st>>>(A, lda, W, M, N, K, C, ldc, P);
  } else {
    const dim3 grid((unsigned)ceil_div(N, 64), (unsigned)ceil_div(M, 64));
    rpp_gemm<4, 4, MODE><<<grid, dim3(256), 0, st>>>(A, lda, W, M, N, K, C, ldc, P);
  }
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// Feed-forward block, fused: x[r] += W2 relu(W1 n[r]). Block (row tile, s)
// takes 32 rows through the s-th of kMlpSplit parts of the hidden width, in
// chunks of 64 through LDS (the hidden activations never leave the compute
// unit), loading the next chunk's weights into registers while the current
// one is used, and writes its partial output; rpp_mlp_sum adds the parts and
// the residual in part order. D = d_model (a multiple of 8, <= 64).
template <int D>
__global__ void __launch_bounds__(256)
rpp_mlp(const float* __restrict__ n, int64_t M, const float* __restrict__ W1,
        const float* __restrict__ W2, int dff, float* __restrict__ part) {
  __shared__ float Ns[kMlpRows][D + 1];
  __shared__ float W1s[kMlpChunk][D + 1];             // hidden unit c of the chunk, its D inputs
  __shared__ float Hs[kMlpRows][kMlpChunk + 1];
  __shared__ float W2s[D][kMlpChunk + 1];             // output o, the chunk's hidden units
  constexpr int OPT = D / 8;                          // outputs per thread
  constexpr int PER = kMlpChunk * D / 256;            // weights of each matrix a thread moves
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kMlpRows;
  const int per_split = (dff + kMlpSplit - 1) / kMlpSplit;
  const int fbeg = min(dff, (int)blockIdx.y * per_split);
  const int fend = min(dff, fbeg + per_split);
  for (int q = t; q < kMlpRows * D; q += 256) {
    const int r = q / D, c = q % D;
    Ns[r][c] = r0 + r < M ? n[(r0 + r) * D + c] : 0.f;
  }
  float w1r[PER], w2r[PER];
  auto fetch = [&](int f0) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = t + 256 * u;
      const int c = q / D, k = q % D;                 // W1 row f0 + c, column k
      w1r[u] = f0 + c < fend ? W1[(int64_t)(f0 + c) * D + k] : 0.f;
      const int o = q / kMlpChunk, kk = q % kMlpChunk;   // W2 row o, column f0 + kk
      w2r[u] = f0 + kk < fend ? W2[(int64_t)o * dff + f0 + kk] : 0.f;
    }
  };
  const int r = t >> 3;                               // this thread's row
  const int c0 = (t & 7) * 8;                         // its 8 hidden units of a chunk
  const int o0 = (t & 7) * OPT;                       // its output columns
  float acc[OPT];
#pragma unroll
  for (int j = 0; j < OPT; ++j) acc[j] = 0.f;
  if (fbeg < fend) fetch(fbeg);
  for (int f0 = fbeg; f0 < fend; f0 += kMlpChunk) {
    __syncthreads();                                  // the previous chunk is fully used
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = t + 256 * u;
      W1s[q / D][q % D] = w1r[u];
      W2s[q / kMlpChunk][q % kMlpChunk] = w2r[u];
    }
    __syncthreads();
    if (f0 + kMlpChunk < fend) fetch(f0 + kMlpChunk);  // in flight during this chunk
    float hv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) hv[j] = 0.f;
#pragma unroll 8
    for (int k = 0; k < D; ++k) {
      const float a = Ns[r][k];
#pragma unroll
      for (int j = 0; j < 8; ++j) hv[j] = fmaf(a, W1s[c0 + j][k], hv[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) Hs[r][c0 + j] = fmaxf(hv[j], 0.f);
    __syncthreads();
#pragma unroll 8
    for (int k = 0; k < kMlpChunk; ++k) {
      const float a = Hs[r][k];
#pragma unroll
      for (int j = 0; j < OPT; ++j) acc[j] = fmaf(a, W2s[o0 + j][k], acc[j]);
    }
  }
  if (r0 + r < M) {
    float* const out = part + ((int64_t)blockIdx.y * M + r0 + r) * D + o0;
#pragma unroll
    for (int j = 0; j < OPT; ++j) out[j] = acc[j];
  }
}

// x += part[0] + part[1] + ... in part order
__global__ void rpp_mlp_sum(const float* __restrict__ part, int64_t n, float* __restrict__ x) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q >= n) return;
  float v = part[q];
#pragma unroll
  for (int s = 1; s < kMlpSplit; ++s) v += part[s * n + q];
  x[q] += v;
}

int mlp(hipStream_t st, const float* n, int64_t M, int d, const float* W1, const float* W2,
        int dff, float* hid, float* x) {
  // hid (M * dff floats) holds the kMlpSplit partial outputs (M * d each)
  const dim3 grid((unsigned)ceil_div(M, kMlpRows), kMlpSplit);
  switch (d) {
    case 16: rpp_mlp<16><<<grid, dim3(256), 0, st>>>(n, M, W1, W2, dff, hid); break;
    case 32: rpp_mlp<32><<<grid, dim3(256), 0, st>>>(n, M, W1, W2, dff, hid); break;
    case 64: rpp_mlp<64><<<grid, dim3(256), 0, st>>>(n, M, W1, W2, dff, hid); break;
    default: {                                        // other widths: two GEMMs via memory
      int rc = gemm<G_RELU>(st, n, d, W1, M, dff, d, hid, dff);
      if (rc != MOE_OK) return rc;
      return gemm<G_ADD>(st, hid, dff, W2, M, d, dff, x, d);
    }
  }
  if (hipGetLastError() != hipSuccess) return MOE_ERR_HIP;
  rpp_mlp_sum<<<dim3((unsigned)ceil_div(M * d, 256)), dim3(256), 0, st>>>(hid, M * d, x);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

template <int MODE>
int rows32(hipStream_t st, const Rows32& a) {
  // 16 rows a block while that leaves a compute unit no more than one block,
  // else 32 rows, which read the weights half as often
  const int64_t b16 = ceil_div(a.M, 16);
  if (b16 <= device_cu_count()) rpp_rows32<MODE, 1, 8><<<dim3((unsigned)b16), dim3(512), 0, st>>>(a);
  else rpp_rows32<MODE, 2, 8><<<dim3((unsigned)ceil_div(a.M, 32)), dim3(512), 0, st>>>(a);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

int attention(hipStream_t st, int dk, const float* Q, int64_t ldq, const float* Kp,
              const float* Vp, int64_t ldkv, int B, int S, int h, const float* rel,
              const RelBuckets& rb, bool use_bias, bool causal, float* O, int64_t ldo) {
  const dim3 grid((unsigned)ceil_div(S, kAttQ), (unsigned)h, (unsigned)B);
  const size_t lds = ((size_t)2 * S * dk + 2 * S) * sizeof(float);
  const size_t lds8 = ((size_t)ceil_div(S, 64) * 64 * 16 + 32 + 2 * (size_t)S) * sizeof(float);
  if (dk == 8 && lds8 <= 64 * 1024) {                // padded keys still fit
    const dim3 grid8((unsigned)ceil_div(S, kAtt8Q), (unsigned)h, (unsigned)B);
    if (use_bias)
      rpp_attention8<true><<<grid8, dim3(kAtt8Threads), lds8, st>>>(
          Q, ldq, Kp, Vp, ldkv, S, h, rel, rb, causal ? 1 : 0, O, ldo);
    else
      rpp_attention8<false><<<grid8, dim3(kAtt8Threads), lds8, st>>>(
          Q, ldq, Kp, Vp, ldkv, S, h, rel, rb, causal ? 1 : 0, O, ldo);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
  }
#define MOE_ATT(DKV)                                                                          \
  rpp_attention<DKV><<<grid, dim3(kAttQ * kSplit), lds, st>>>(                               \
      Q, ldq, Kp, Vp, ldkv, S, h, rel, rb, use_bias ? 1 : 0, causal ? 1 : 0, O, ldo)
  switch (dk) {
    case 4: MOE_ATT(4); break;
    case 8: MOE_ATT(8); break;
    case 16: MOE_ATT(16); break;
    case 32: MOE_ATT(32); break;
    case 64: MOE_ATT(64); break;
    default: return MOE_ERR_UNSUPPORTED;
  }
#undef MOE_ATT
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

}  // namespace
}  // namespace moe

extern "C" size_t moe_rpp_weights_count(const moe_rpp_dims* dims) {
  if (!moe::dims_ok(dims)) return 0;
  return moe::rpp_offsets(*dims).total;
}

extern "C" size_t moe_rpp_workspace(int32_t B, int32_t S, const moe_rpp_dims* dims) {
  if (!moe::dims_ok(dims) || B < 1 || S < 1) return 0;
  return moe::rpp_ws((int64_t)B * S, *dims).total;
}

extern "C" int moe_rpp_forward(const int32_t* ids, int32_t B, int32_t S, const moe_rpp_dims* dims,
                               const float* weights, float* probs, float* logits, int32_t* err,
                               void* workspace, size_t ws_bytes, void* stream) {
  using namespace moe;
  MOE_CHECK_ARG(ids && weights && probs && err && dims_ok(dims) && B >= 1 && S >= 1);
  const moe_rpp_dims g = *dims;
  const int d = g.d_model, h = g.n_heads, dk = d / h;
  const int64_t M = (int64_t)B * S;
  if (M * std::max(g.d_ff, 3 * d) >= ((int64_t)1 << 31) / 4 ||
      ((size_t)2 * S * dk + 2 * S) * sizeof(float) > 64 * 1024)
    return MOE_ERR_UNSUPPORTED;
  RelBuckets rb_enc{}, rb_dec{};
  if (!make_buckets(true, g.num_buckets, g.max_distance, &rb_enc) ||
      !make_buckets(false, g.num_buckets, g.max_distance, &rb_dec))
    return MOE_ERR_UNSUPPORTED;
  const RppWs lay = rpp_ws(M, g);
  if (!workspace || ws_bytes < lay.total || (reinterpret_cast<uintptr_t>(workspace) & 255))
    return MOE_ERR_WORKSPACE;
  char* ws = static_cast<char*>(workspace);
  auto F = [&](size_t off) { return reinterpret_cast<float*>(ws + off); };
  float *x = F(lay.x), *y = F(lay.y), *n = F(lay.n), *enc = F(lay.enc), *o = F(lay.o);
  float *qkv = F(lay.qkv), *kv = F(lay.kv), *hid = F(lay.hid);
  float* lg = logits ? logits : F(lay.logits);
  const RppOffsets wo = rpp_offsets(g);
  const float* W = weights;
  hipStream_t st = as_stream(stream);
  const dim3 rows((unsigned)ceil_div(M * 32, 256));      // 32 lanes per row
  const size_t dd = (size_t)d * d, df = (size_t)d * g.d_ff;
  int rc = MOE_OK;
#define MOE_RC(expr)                  \
  do {                                \
    rc = (expr);                      \
    if (rc != MOE_OK) return rc;      \
  } while (0)

  // Hidden size 32: one launch per attention and one for all between two of
  // them. Needs a layer on each side, and 16-byte aligned weight rows (the
  // bias tables keep them so: num_buckets is a power of two from 4 on).
  if (d == 32 && g.n_enc >= 1 && g.n_dec >= 1 && g.d_ff % 4 == 0 &&
      (reinterpret_cast<uintptr_t>(weights) & 15) == 0) {
    Rows32 a{};
    a.M = M;
    a.eps = g.eps;
    a.ids = ids;
    a.emb = W + wo.emb;
    a.vocab = g.vocab;
    a.err = err;
    a.o = o;
    a.dff = g.d_ff;
    auto embed = [&](float* stream_x, const float* layer) {
      a.x = stream_x;
      a.ln = layer;
      a.wnext = layer + d;
      a.n_next = 3 * d;
      a.next = qkv;
      return rows32<kRowsEmbed>(st, a);
    };
    // feed-forward at p (norm, W1, W2), then the next layer's first norm and
    // projection, or the stack's last norm into `last`
    auto feed_forward = [&](const float* wout, const float* p, const float* next_layer,
                            const float* ln_last, float* last) {
      a.wout = wout;
      a.ln = p;
      a.w1 = p + d;
      a.w2 = a.w1 + df;
      a.ln_next = next_layer ? next_layer : ln_last;
      a.wnext = next_layer ? next_layer + d : nullptr;
      a.n_next = next_layer ? 3 * d : 0;
      a.next = next_layer ? qkv : last;
      return rows32<kRowsMlp>(st, a);
    };
    MOE_RC(embed(x, W + wo.enc[0]));
    for (int l = 0; l < g.n_enc; ++l) {
      const float* const wout = W + wo.enc[l] + d + 3 * dd;
      MOE_RC(attention(st, dk, qkv, 3 * d, qkv + d, qkv + 2 * d, 3 * d, B, S, h, W + wo.enc_rel,
                       rb_enc, true, false, o, d));
      MOE_RC(feed_forward(wout, wout + dd, l + 1 < g.n_enc ? W + wo.enc[l + 1] : nullptr,
                          W + wo.enc_ln, enc));
    }
    MOE_RC(embed(y, W + wo.dec[0]));
    for (int l = 0; l < g.n_dec; ++l) {
      const float* const wout = W + wo.dec[l] + d + 3 * dd;
      const float* const ln2 = wout + dd;
      const float *cq = ln2 + d, *ckv = cq + dd, *cout = ckv + 2 * dd;
      MOE_RC(attention(st, dk, qkv, 3 * d, qkv + d, qkv + 2 * d, 3 * d, B, S, h, W + wo.dec_rel,
                       rb_dec, true, true, o, d));
      a.wout = wout;
      a.ln = ln2;
      a.wnext = cq;
      a.n_next = d;
      a.next = qkv;
      a.enc = enc;
      a.wkv = ckv;
      a.kv = kv;
      MOE_RC(rows32<kRowsCross>(st, a));
      MOE_RC(attention(st, dk, qkv, d, kv, kv + d, 2 * d, B, S, h, nullptr, rb_dec, false, false,
                       o, d));
      MOE_RC(feed_forward(cout, cout + dd, l + 1 < g.n_dec ? W + wo.dec[l + 1] : nullptr,
                          W + wo.dec_ln, n));
    }
    MOE_RC(gemm<G_SIGMOID>(st, n, d, W + wo.heads, M, (int64_t)g.L * g.E, d, lg,
                           (int64_t)g.L * g.E, probs));
    return MOE_OK;
  }

  rpp_embed<<<dim3((unsigned)ceil_div(M * d, 256)), dim3(256), 0, st>>>(ids, M, g.vocab, d,
                                                                      W + wo.emb, x, err);
  MOE_CHECK_LAUNCH();
  for (int l = 0; l < g.n_enc; ++l) {
    const float* p = W + wo.enc[l];
    const float *ln1 = p, *wqkv = p + d, *wout = wqkv + 3 * dd, *ln2 = wout + dd;
    const float *wi = ln2 + d, *wo2 = wi + df;
    rpp_rmsnorm<<<rows, dim3(256), 0, st>>>(x, M, d, ln1, g.eps, n);
    MOE_CHECK_LAUNCH();
    MOE_RC(gemm<G_STORE>(st, n, d, wqkv, M, 3 * d, d, qkv, 3 * d));
    MOE_RC(attention(st, dk, qkv, 3 * d, qkv + d, qkv + 2 * d, 3 * d, B, S, h, W + wo.enc_rel,
                     rb_enc, true, false, o, d));
    MOE_RC(gemm<G_ADD>(st, o, d, wout, M, d, d, x, d));
    rpp_rmsnorm<<<rows, dim3(256), 0, st>>>(x, M, d, ln2, g.eps, n);
    MOE_CHECK_LAUNCH();
    MOE_RC(mlp(st, n, M, d, wi, wo2, g.d_ff, hid, x));
  }
  rpp_rmsnorm<<<rows, dim3(256), 0, st>>>(x, M, d, W + wo.enc_ln, g.eps, enc);
  MOE_CHECK_LAUNCH();
  rpp_embed<<<dim3((unsigned)ceil_div(M * d, 256)), dim3(256), 0, st>>>(ids, M, g.vocab, d,
                                                                      W + wo.emb, y, err);
  MOE_CHECK_LAUNCH();
  for (int l = 0; l < g.n_dec; ++l) {
    const float* p = W + wo.dec[l];
    const float *ln1 = p, *wqkv = p + d, *wout = wqkv + 3 * dd, *ln2 = wout + dd;
    const float *cq = ln2 + d, *ckv = cq + dd, *cout = ckv + 2 * dd, *ln3 = cout + dd;
    const float *wi = ln3 + d, *wo2 = wi + df;
    rpp_rmsnorm<<<rows, dim3(256), 0, st>>>(y, M, d, ln1, g.eps, n);
    MOE_CHECK_LAUNCH();
    MOE_RC(gemm<G_STORE>(st, n, d, wqkv, M, 3 * d, d, qkv, 3 * d));
    MOE_RC(attention(st, dk, qkv, 3 * d, qkv + d, qkv + 2 * d, 3 * d, B, S, h, W + wo.dec_rel,
                     rb_dec, true, true, o, d));
    MOE_RC(gemm<G_ADD>(st, o, d, wout, M, d, d, y, d));
    rpp_rmsnorm<<<rows, dim3(256), 0, st>>>(y, M, d, ln2, g.eps, n);
    MOE_CHECK_LAUNCH();
    MOE_RC(gemm<G_STORE>(st, n, d, cq, M, d, d, qkv, d));
    MOE_RC(gemm<G_STORE>(st, enc, d, ckv, M, 2 * d, d, kv, 2 * d));
    MOE_RC(attention(st, dk, qkv, d, kv, kv + d, 2 * d, B, S, h, nullptr, rb_dec, false, false,
                     o, d));
    MOE_RC(gemm<G_ADD>(st, o, d, cout, M, d, d, y, d));
    rpp_rmsnorm<<<rows, dim3(256), 0, st>>>(y, M, d, ln3, g.eps, n);
    MOE_CHECK_LAUNCH();
    MOE_RC(mlp(st, n, M, d, wi, wo2, g.d_ff, hid, y));
  }
  rpp_rmsnorm<<<rows, dim3(256), 0, st>>>(y, M, d, W + wo.dec_ln, g.eps, n);
  MOE_CHECK_LAUNCH();
  MOE_RC(gemm<G_SIGMOID>(st, n, d, W + wo.heads, M, (int64_t)g.L * g.E, d, lg,
                         (int64_t)g.L * g.E, probs));
#undef MOE_RC
  return MOE_OK;
}
