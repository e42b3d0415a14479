// Prefill similarity matching (Method section, "Similarity Matching",
// Eqs. 1-3): over a window of the prompt, the accumulative attention score F
// of every head of both models (Eq. 1), each head's TopK token set, and for
// every large head the small head whose TopK set has the largest Jaccard
// similarity (Eqs. 2-3).
//
// The TopK sets and the argmax are integer decisions taken on fp32 sums, so
// every value feeding them has one defined evaluation, the one smallkv.h
// states: logits as sequential fp32 FMA chains; an exp by Cody-Waite
// reduction and a degree-7 Taylor polynomial; row sums and column sums taken
// one term at a time in ascending token order.  The result is bit-exact
// against any implementation of that definition.
//
// Two kernels:
//   match_heads -- one workgroup per head.  The window's query rows are walked
//                  kRows at a time, so that the whole of Eq. 1 stays in the
//                  workgroup: the rows' logits on the matrix cores into LDS,
//                  each row's maximum and exponentials, its sum Z_u (v
//                  ascending), and every column's sum F_v (one thread per
//                  token, u ascending over the row blocks) in a register;
//                  then the TopK set by one wave, which finds the k-th largest
//                  sum bit by bit;
//   match_map   -- one wave per large head: Jaccard ratios against every
//                  small head from TopK bitsets (popcounts), the argmax by
//                  exact cross-multiplication, ties to the lowest small head.
//
// The logits are fp32 FMA chains, and v_mfma_f32_16x16x1 (K = 1: one product
// per element and instruction) is exactly one step of 16 x 64 of them: D =
// fma(A, B, C) with one rounding, subnormals, infinities and NaN included
// (compared bit for bit with the vector FMA over arbitrary bit patterns).  It
// runs at 140-150 TFLOP/s here against 75 for plain vector FMAs.
#include "common.h"
#include "launch.h"

#pragma clang fp contract(off)

namespace smallkv {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int kMatchThreads = 256;
constexpr int kWaves = kMatchThreads / kWave;
constexpr int kXcd = 8;
constexpr int kMaxWin = 256;          // tokens per window at most (one thread per token)
constexpr int kStrip = 16;            // query rows per MFMA
constexpr int kCols = 64;             // tokens per MFMA (4 blocks of 16)
constexpr int kSlice = 32;            // head dims of the operands loaded at a time
constexpr int kRows = 2 * kStrip;     // query rows per pass

struct HeadsArgs {
  const void *q, *k;  // [B][layers][hq][w_cap][d], [B][layers][hkv][w_cap][d]
  int layers, hq, hkv, d, heads, head0;  // heads of this model, the first one's index of H
  float scale;
};

struct MatchArgs {
  HeadsArgs m[2];           // the heads of this launch: m[0]'s, then m[1]'s (heads 0: none)
  int w_cap, H, nw;         // nw: 64-token words per TopK bitset
  const int32_t *win_len, *top_k;
  uint64_t *bits;           // [B][H][nw]
  float *scores;            // optional [B][H][w_cap]
  uint64_t *top_bits;       // optional copy of bits
};

// Workgroups an XCD (x % 8) takes of n heads: consecutive ones, so that the
// query heads of a kv head read its keys through one L2.
__host__ __device__ constexpr int per_xcd(int n) { return (n + kXcd - 1) / kXcd; }

// The operands of one (16 query rows x 64 tokens) tile over kSlice dims, as
// loaded: lane l holds dims 8*(l/16) .. +7 of query row l%16 (so block b of
// the A operand holds dims 8b..) and all the slice's dims of token l.
template <typename T>
struct Raw {
  static constexpr int per = elem<T>::per16;
  uint4 q[kSlice / 4 / per], k[kSlice / per];
};

template <typename T>
__device__ __forceinline__ void load_raw(Raw<T> &r, const T *Q, const T *K, int d, int w, int u0,
                                         int v0, int c0) {
  const int lane = threadIdx.x & (kWave - 1);
  // rows past the window repeat its last one: their logits are not used
  const T *q = Q + min(u0 + (lane & 15), w - 1) * d + c0 + (lane >> 4) * (kSlice / 4);
  const T *k = K + min(v0 + lane, w - 1) * d + c0;
#pragma unroll
  for (int i = 0; i < kSlice / 4 / Raw<T>::per; ++i) r.q[i] = reinterpret_cast<const uint4 *>(q)[i];
#pragma unroll
  for (int i = 0; i < kSlice / Raw<T>::per; ++i) r.k[i] = reinterpret_cast<const uint4 *>(k)[i];
}

// One chain step of the tile for each dim of block BLK (8 dims), ascending.
template <typename T, int BLK>
__device__ __forceinline__ void chain8(f32x16_t &acc, const Raw<T> &r, const float (&a)[kSlice / 4]) {
  constexpr int per = Raw<T>::per;
#pragma unroll
  for (int i = 0; i < 8 / per; ++i) {
    float kv[per];
    elem<T>::unpack(r.k[BLK * 8 / per + i], kv);
#pragma unroll
    for (int j = 0; j < per; ++j)
      acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a[i * per + j], kv[j], acc, 2, BLK, 0);
  }
}

template <typename T>
__device__ __forceinline__ void chain_slice(f32x16_t &acc, const Raw<T> &r) {
  float a[kSlice / 4];
#pragma unroll
  for (int i = 0; i < kSlice / 4 / Raw<T>::per; ++i) elem<T>::unpack(r.q[i], a + i * Raw<T>::per);
  chain8<T, 0>(acc, r, a);
  chain8<T, 1>(acc, r, a);
  chain8<T, 2>(acc, r, a);
  chain8<T, 3>(acc, r, a);
}

template <int CTRL>
__device__ __forceinline__ float dpp_max(float x) {
  return fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, false)));
}

// Maxima over the wave of eight values at once: halving exchanges hand every
// eight lanes one of them, which they then reduce.  Value i's maximum ends in
// lanes 8i .. 8i+7.
__device__ __forceinline__ float wave_max8(float (&v)[8]) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // lanes 0-31 keep values 0-3
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 4]), false, false);
    v[i] = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // even 16-lane rows keep the lower two
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 2]), false, false);
    v[i] = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  const bool upper = (lane & 8) != 0;
  const float keep = upper ? v[1] : v[0], send = upper ? v[0] : v[1];
  float x = fmaxf(keep, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(send), 0x128, 0xf, 0xf, false)));
  x = dpp_max<0xB1>(x);     // lane ^ 1
  x = dpp_max<0x4E>(x);     // lane ^ 2
  return dpp_max<0x141>(x); // 8-lane mirror
}

// Exponentials, and with them Z and F, are held scaled by 2^64 (exact, as
// none of them is ever subnormal or near overflow: e is 0 or 2^-116 .. 1), so
// that no remainder of the divisions is subnormal.
// LDS of a workgroup (floats): the pass's logits [kRows][pitch], then Z and
// its reciprocal per row.  The column sums take the logits' place at the end.
// The pitch follows the window capacity, so that five workgroups of 200-token
// windows fit a CU.
__host__ __device__ constexpr int pitch_of(int w_cap) { return (w_cap + 3) / 4 * 4 + 4; }
constexpr size_t heads_lds(int w_cap) {
  const size_t f = (size_t)kRows * pitch_of(w_cap);
  return ((f > kMaxWin ? f : kMaxWin) + 4 * kRows) * sizeof(float);
}

// Bound by the SIMDs' issue: fp32 MFMAs and vector instructions do not overlap
// (measured side by side: their times add), and the window of the Qwen2 pair
// (784 heads of d 128 and 336 of d 64, 200 tokens) has 106k cycles per SIMD of
// the one (7.1 GFLOP of tiles for 4.9 of logits) and 90k of the other; the
// rest is the passes' barriers, hidden by five workgroups per CU (three take
// 164 us, two 207).  Whole matching 249 us with the logits in memory between
// kernels and vector FMAs, 131 like this.
template <typename T>
__device__ __forceinline__ void head_scores(const MatchArgs &a, const HeadsArgs &m, float *lds,
                                            int j, int b) {
  const int pitch = pitch_of(a.w_cap);
  float *const s = lds;
  float4 *const zr = reinterpret_cast<float4 *>(lds + max(kRows * pitch, kMaxWin));
  const int lane = threadIdx.x & (kWave - 1);
  // the wave's part, shifted between workgroups: waves of one index share a
  // SIMD, and the first parts have more of the tiles and columns (131 us
  // against 135 without the shift on the 200-token Qwen2 pair; giving every
  // wave the same number of tiles instead: 135)
  const int part = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + blockIdx.x / kXcd) & (kWaves - 1);
  const int w = clampi(a.win_len[b], 1, a.w_cap);
  const int layer = j / m.hq, h = j % m.hq, g = h / (m.hq / m.hkv);
  const T *Q = static_cast<const T *>(m.q) + (((int64_t)b * m.layers + layer) * m.hq + h) * a.w_cap * m.d;
  const T *K = static_cast<const T *>(m.k) + (((int64_t)b * m.layers + layer) * m.hkv + g) * a.w_cap * m.d;
  const int64_t hrow = (int64_t)b * a.H + m.head0 + j;
  const int c0 = part * kCols, col = c0 + lane;  // the wave's 64 columns of F
  float f = 0.0f;
  // tiles of the pass from row r0: 64-token chunks of one strip, then of the next
  auto chunks = [&](int r0) { return (min(r0 + kRows, w) + kCols - 1) / kCols; };
  auto tiles_of = [&](int r0) { return w - r0 > kStrip ? 2 * chunks(r0) : chunks(r0); };
  auto load_tile = [&](Raw<T> &r, int r0, int tile, int c) {
    const int nch = chunks(r0), strip = tile >= nch ? 1 : 0;
    load_raw<T>(r, Q, K, m.d, w, r0 + strip * kStrip, (tile - strip * nch) * kCols, c);
  };
  auto load_first = [&](Raw<T> &r, int r0) {  // the wave's first tile of a pass
    if (r0 < w && part < tiles_of(r0)) load_tile(r, r0, part, 0);
  };
  Raw<T> x, y;  // two slices: one in use, the next on its way
  load_first(x, 0);
  for (int r0 = 0; r0 < w; r0 += kRows) {
    const int nr = min(kRows, w - r0);
    // ---- logits: (16 rows x 64 tokens) tiles, one at a time per wave ------
    const int nch = chunks(r0), tiles = tiles_of(r0);
    for (int tile = part; tile < tiles; tile += kWaves) {
      f32x16_t acc = {};
      for (int c = 0; c < m.d; c += 2 * kSlice) {
        load_tile(y, r0, tile, c + kSlice);
        chain_slice<T>(acc, x);
        if (c + 2 * kSlice < m.d) load_tile(x, r0, tile, c + 2 * kSlice);
        else if (tile + kWaves < tiles) load_tile(x, r0, tile + kWaves, 0);
        else load_first(x, r0 + kRows);
        chain_slice<T>(acc, y);
      }
      // lane l: rows 4(l/16) + r, tokens 16 blk + l%16 of the tile (tokens past
      // the row's pitch go to its last, unused column)
      const int strip = tile >= nch ? 1 : 0, v0 = (tile - strip * nch) * kCols;
      const int row0 = strip * kStrip + (lane >> 4) * 4, vl = v0 + (lane & 15);
      float *const srow = s + row0 * pitch;
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        float *const p = srow + min(vl + blk * 16, pitch - 1);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          p[r * pitch] = __builtin_fmaf(acc[4 * blk + r], m.scale, 0.0f);  // (a zero's sign is not used)
      }
    }
    if (part >= tiles) load_first(x, r0 + kRows);
    __syncthreads();
    // ---- row maxima, then exponentials in place; 0 past the diagonal (adds
    // nothing to Z)
    constexpr int kOwn = kRows / kWaves;
    const int own = part * kOwn;
    if (own < nr) {  // the wave's rows (past nr: old values, not used)
      float e[kOwn], mx[kOwn];
      auto chunk = [&](int ch) {
        const float *p = s + own * pitch + min(ch * kCols + lane, pitch - 1);
#pragma unroll
        for (int i = 0; i < kOwn; ++i) e[i] = p[i * pitch];
        if (ch * kCols + kCols > r0 + 1) {  // (uniform) the chunk meets the diagonal
          const int lim = r0 + own - ch * kCols - lane;
#pragma unroll
          for (int i = 0; i < kOwn; ++i) e[i] = lim + i >= 0 ? e[i] : -INFINITY;
        }
      };
#pragma unroll
      for (int i = 0; i < kOwn; ++i) mx[i] = -INFINITY;
#pragma unroll 1
      for (int ch = 0; ch < nch; ++ch) {
        chunk(ch);
#pragma unroll
        for (int i = 0; i < kOwn; ++i) mx[i] = fmaxf(mx[i], e[i]);
      }
      static_assert(kOwn == 8, "wave_max8");
      const float red = wave_max8(mx);
#pragma unroll
      for (int i = 0; i < kOwn; ++i)
        mx[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(red), 8 * i));
#pragma unroll 1
      for (int ch = 0; ch < nch; ++ch) {
        chunk(ch);
        float *p = s + own * pitch + min(ch * kCols + lane, pitch - 1);
#pragma unroll
        for (int i = 0; i < kOwn; ++i) p[i * pitch] = exp_up(e[i] - mx[i]);
      }
    }
    __syncthreads();
    // ---- Z_u: one thread per row, v ascending -------------------------------
    if (part == kWaves - 1 && lane < nr) {
      float z = 0.0f;
      const float4 *row = reinterpret_cast<const float4 *>(s + lane * pitch);
      const int n4 = (r0 + nr + 3) / 4;
      auto add4 = [&](const float4 &e) {
        z = z + e.x;
        z = z + e.y;
        z = z + e.z;
        z = z + e.w;
      };
      int i = 0;
      for (; i + 4 <= n4; i += 4) {  // four reads in flight
        const float4 e0 = row[i], e1 = row[i + 1], e2 = row[i + 2], e3 = row[i + 3];
        add4(e0);
        add4(e1);
        add4(e2);
        add4(e3);
      }
      for (; i < n4; ++i) add4(row[i]);
      const Recip r = recip(z * kDown);
      zr[lane] = make_float4(r.z, r.y, r.dy, 0.0f);
    }
    __syncthreads();
    // ---- F_v: one thread per token, u ascending ---------------------------
    if (c0 < r0 + nr && col < w) {
      constexpr int kBatch = 8;
      const bool below = c0 + kCols <= r0 + 1;  // (uniform) the columns are below every row
      const float *scol = s + col;
      for (int i = 0; i < nr; i += kBatch) {  // rows past nr hold old values and are not added
        float p[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
          const float4 z = zr[i + q];
          p[q] = div_by(scol[(i + q) * pitch], Recip{z.x, z.y, z.z});
        }
        if (below && i + kBatch <= nr) {
#pragma unroll
          for (int q = 0; q < kBatch; ++q) f = f + p[q];
        } else {
#pragma unroll
          for (int q = 0; q < kBatch; ++q)
            if (i + q < nr && col <= r0 + i + q) f = f + p[q];
        }
      }
    }
    __syncthreads();  // before the next pass writes its logits
  }
  f *= kDown;
  s[col] = f;
  __syncthreads();
  if (a.scores && col < w) a.scores[hrow * a.w_cap + col] = f;
  // ---- TopK: ranked first by larger F, then by lower token index ----------
  // One wave holds all the sums (their bits order as they do) and finds the
  // k-th largest bit by bit; a NaN (of infinite logits) ranks above nothing
  // and below nothing, and so is in.
  if (part != 0) return;
  constexpr int kWords = kMaxWin / kWave;
  const int k = clampi(a.top_k[b], 1, w);
  uint32_t key[kWords];
  uint64_t valid[kWords];
#pragma unroll
  for (int c = 0; c < kWords; ++c) {
    const float x = s[c * kWave + lane];
    valid[c] = __builtin_amdgcn_ballot_w64(c * kWave + lane < w && x == x);
    key[c] = __builtin_amdgcn_inverse_ballot_w64(valid[c]) ? __float_as_uint(x) : 0u;
  }
  uint32_t kth = 0;
  for (uint32_t bit = 1u << 30; bit; bit >>= 1) {
    const uint32_t cand = kth | bit;
    int n = 0;
#pragma unroll
    for (int c = 0; c < kWords; ++c) n += __popcll(__builtin_amdgcn_ballot_w64(key[c] >= cand));
    if (n >= k) kth = cand;
    if (n == k) break;
  }
  int need = k, before = 0;  // ties taken, from the lowest token on
#pragma unroll
  for (int c = 0; c < kWords; ++c) need -= __popcll(__builtin_amdgcn_ballot_w64(key[c] > kth));
#pragma unroll
  for (int c = 0; c < kWords; ++c) {
    const uint64_t ties = __builtin_amdgcn_ballot_w64(key[c] == kth) & valid[c];
    const int rank = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(ties >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)ties, 0));
    const uint64_t word = __builtin_amdgcn_ballot_w64(key[c] > kth) |
                          (ties & __builtin_amdgcn_ballot_w64(rank < need)) |
                          (__builtin_amdgcn_ballot_w64(c * kWave + lane < w) & ~valid[c]);
    if (lane == 0 && c < a.nw) {
      a.bits[hrow * a.nw + c] = word;
      if (a.top_bits) a.top_bits[hrow * a.nw + c] = word;
    }
    before += __popcll(ties);
  }
}

// blockIdx.x: a head of either model, m[0]'s (the larger ones) first: the
// launch's last workgroups are its shortest; blockIdx.y: the sequence.
template <typename T>
__global__ __launch_bounds__(kMatchThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 5)))
void match_heads(MatchArgs a) {
  extern __shared__ __align__(16) float lds[];
  const int xcd = blockIdx.x % kXcd, y = blockIdx.x / kXcd;
  const int n0 = per_xcd(a.m[0].heads), n1 = per_xcd(a.m[1].heads);
  const int mi = y >= n0 ? 1 : 0;
  const HeadsArgs &m = a.m[mi];
  const int j = mi ? xcd * n1 + (y - n0) : xcd * n0 + y;
  if (j >= m.heads) return;  // (padding)
  head_scores<T>(a, m, lds, j, blockIdx.y);
}

struct MapArgs {
  const uint64_t *bits;
  int H, nl, ns, nw;
  int32_t *head_map;  // [B][nl]
};

// a/b > c/d for b, d > 0 (a may be -1 as "no candidate")
__device__ __forceinline__ bool ratio_gt(int a, int b, int c, int d) { return a * d > c * b; }

__global__ __launch_bounds__(kMatchThreads) void match_map(MapArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int i = blockIdx.x * (kMatchThreads / kWave) + threadIdx.x / kWave;
  const int b = blockIdx.y;
  if (i >= a.nl) return;  // whole waves; no barrier follows
  const uint64_t *Ti = a.bits + ((int64_t)b * a.H + i) * a.nw;
  uint64_t ti[4];
  int ci = 0;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    ti[x] = x < a.nw ? Ti[x] : 0ull;
    ci += __popcll(ti[x]);
  }
  int bn = -1, bd = 1, bj = 0x7fffffff;
  for (int j = lane; j < a.ns; j += kWave) {
    const uint64_t *Tj = a.bits + ((int64_t)b * a.H + a.nl + j) * a.nw;
    int in = 0, cj = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const uint64_t tj = x < a.nw ? Tj[x] : 0ull;
      in += __popcll(ti[x] & tj);
      cj += __popcll(tj);
    }
    const int un = ci + cj - in;
    if (ratio_gt(in, un, bn, bd)) {  // j rises: a tie keeps the lower one
      bn = in;
      bd = un;
      bj = j;
    }
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const int n2 = __shfl_xor(bn, o, kWave), d2 = __shfl_xor(bd, o, kWave);
    const int j2 = __shfl_xor(bj, o, kWave);
    if (ratio_gt(n2, d2, bn, bd) || (n2 * bd == bn * d2 && j2 < bj)) {
      bn = n2;
      bd = d2;
      bj = j2;
    }
  }
  if (lane == 0) a.head_map[(int64_t)b * a.nl + i] = bj;
}

HeadsArgs heads_of(const smallkv_window_t &m, int head0) {
  HeadsArgs h{};
  h.q = m.q;
  h.k = m.k;
  h.layers = m.n_layers;
  h.hq = m.n_q_heads;
  h.hkv = m.n_kv_heads;
  h.d = m.head_dim;
  h.heads = m.n_layers * m.n_q_heads;
  h.head0 = head0;
  h.scale = m.scale;
  return h;
}

hipError_t launch_heads(const MatchArgs &a, int batch, bool f32, hipStream_t st) {
  const dim3 grid(kXcd * (per_xcd(a.m[0].heads) + per_xcd(a.m[1].heads)), batch);
  const size_t lds = heads_lds(a.w_cap);
  if (f32)
    hipLaunchKernelGGL((match_heads<float>), grid, dim3(kMatchThreads), lds, st, a);
  else
    hipLaunchKernelGGL((match_heads<bf16_t>), grid, dim3(kMatchThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace

MatchLayout match_layout(const smallkv_match_t &m) {
  MatchLayout l{};
  const int64_t H = (int64_t)m.large.n_layers * m.large.n_q_heads +
                    (int64_t)m.small.n_layers * m.small.n_q_heads;
  l.nw = (m.w_cap + kWave - 1) / kWave;
  // Only the bitsets at the start are used (the logits stay in LDS).  The size
  // is that of one logit matrix, its tile maxima and row statistics before them,
  // as callers that keep a workspace were told.
  auto round256 = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t rows = (size_t)m.batch * H * m.w_cap, ld = (m.w_cap + 3) / 4 * 4, nt = l.nw;
  l.total = round256(rows * ld * sizeof(float)) + round256(rows * nt * sizeof(float)) +
            round256(rows * sizeof(float2)) + (size_t)m.batch * H * l.nw * sizeof(uint64_t);
  return l;
}

hipError_t launch_match(const smallkv_match_t &m, void *ws, hipStream_t st) {
  uint64_t *bits = static_cast<uint64_t *>(ws);
  const int nl = m.large.n_layers * m.large.n_q_heads;
  const int ns = m.small.n_layers * m.small.n_q_heads;
  MatchArgs a{};
  a.w_cap = m.w_cap;
  a.H = nl + ns;
  a.nw = match_layout(m).nw;
  a.win_len = m.win_len;
  a.top_k = m.top_k;
  a.bits = bits;
  a.scores = m.scores;
  a.top_bits = m.top_bits;
  a.m[0] = heads_of(m.large, 0);
  hipError_t e;
  if (m.small.dtype == m.large.dtype) {  // both models in one launch
    a.m[1] = heads_of(m.small, nl);
    e = launch_heads(a, m.batch, m.large.dtype == SMALLKV_F32, st);
  } else {
    e = launch_heads(a, m.batch, m.large.dtype == SMALLKV_F32, st);
    if (e != hipSuccess) return e;
    a.m[0] = heads_of(m.small, nl);
    e = launch_heads(a, m.batch, m.small.dtype == SMALLKV_F32, st);
  }
  if (e != hipSuccess) return e;
  MapArgs ma{bits, a.H, nl, ns, a.nw, m.head_map};
  hipLaunchKernelGGL(match_map, dim3((nl + kWaves - 1) / kWaves, m.batch), dim3(kMatchThreads), 0, st,
                     ma);
  return hipGetLastError();
}

}  // namespace smallkv
