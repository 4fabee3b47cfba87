// Backward of a submanifold sparse convolution layer (chain rule on the forward definition).
//   dZ = dY * [Y > 0] (ReLU'(0) = 0) or dY;
//   dX = conv(dZ, W'), W'_k = (W_{26-k})^T: the rulebook is symmetric (R_{26-k} is R_k with the
//        roles of input and output swapped), so the data gradient is a forward convolution;
//   dW_k = sum_{(i,r) in R_k} X[i]^T dZ[r]: per-offset reduced outer products over the CSR
//        pair list, cut into a fixed number of slices per offset and reduced in a fixed order;
//   db = sum_r dZ[r], from per-row-block partial sums written while dZ is formed.
// Every float32 reduction adds short plain partial sums into a Neumaier-compensated total, and
// all reduction orders are fixed, so gradients are bit-identical run to run.
#include <type_traits>

#include "bwd_layout.hpp"

namespace npvs {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;


struct Comp {  // Neumaier-compensated float sum
  float s, c;
  __device__ __forceinline__ void add(float y) {
    float t = s + y;
    c += (__builtin_fabsf(s) >= __builtin_fabsf(y)) ? (s - t) + y : (y - t) + s;
    s = t;
  }
  __device__ __forceinline__ void merge(const Comp &o) {
    add(o.s);
    c += o.c;
  }
  __device__ __forceinline__ float value() const { return s + c; }
};

__device__ __forceinline__ float load_as_f32(const float *p, int64_t i) { return p[i]; }
__device__ __forceinline__ float load_as_f32(const uint16_t *p, int64_t i) { return bf16_to_f32(p[i]); }

constexpr int kDbBlocks = kBwdDbBlocks;  // row blocks of the bias-gradient partial sums (one layer)

// dZ in float32 (for wgrad; nullable) and, for the BF16 path, a bfloat16 copy (MFMA operand),
// plus the bias-gradient partial of this block's rows: blockIdx.x = partial row, blockIdx.y = a
// window of 64 columns (one window when C <= 64), 256 threads.  With vec (C % 4 == 0 and 16-byte
// aligned rows) a thread owns 4 adjacent columns, else one; the threads of a row group cover the
// window of one row, the row groups stride over the block's rows and are combined in LDS in a
// fixed order.
__device__ __forceinline__ void load4(const float *p, int64_t e, float *v) {
  const f32x4_t x = *reinterpret_cast<const f32x4_t *>(p + e);
  v[0] = x[0], v[1] = x[1], v[2] = x[2], v[3] = x[3];
}
__device__ __forceinline__ void load4(const uint16_t *p, int64_t e, float *v) {
  const uint2 x = *reinterpret_cast<const uint2 *>(p + e);
  v[0] = bf16_to_f32((uint16_t)x.x), v[1] = bf16_to_f32((uint16_t)(x.x >> 16));
  v[2] = bf16_to_f32((uint16_t)x.y), v[3] = bf16_to_f32((uint16_t)(x.y >> 16));
}

template <typename T>
__global__ __launch_bounds__(256) void relu_grad_kernel(const T *__restrict__ Y, const float *__restrict__ dY,
                                                         const npvs_counts *__restrict__ counts, int C, int relu,
                                                         int vec, float *__restrict__ dZ32, uint16_t *__restrict__ dZ16,
                                                         float *__restrict__ dbpart) {
  __shared__ float red[256 * 4];
  const int64_t n = counts->n_sites;
  const int64_t r0 = n * blockIdx.x / gridDim.x, r1 = n * (blockIdx.x + 1) / gridDim.x;
  const int c0 = 64 * blockIdx.y, Cw = C - c0 < 64 ? C - c0 : 64;
  const int V = vec ? 4 : 1, TPR = Cw / V, RG = 256 / TPR;
  const int cg = threadIdx.x % TPR, rg = threadIdx.x / TPR;
  Comp a[4] = {{0.0f, 0.0f}, {0.0f, 0.0f}, {0.0f, 0.0f}, {0.0f, 0.0f}};
  if (rg < RG) {
    if (vec) {
      for (int64_t r = r0 + rg; r < r1; r += RG) {
        const int64_t e = r * C + c0 + 4 * cg;
        float g[4], y[4];
        load4(dY, e, g);
        if (relu) {
          load4(Y, e, y);
#pragma unroll
          for (int i = 0; i < 4; ++i) g[i] = y[i] > 0.0f ? g[i] : 0.0f;
        }
        f32x4_t o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          o[i] = g[i];
          a[i].add(g[i]);
        }
        if (dZ32) *reinterpret_cast<f32x4_t *>(dZ32 + e) = o;
        if (dZ16) {
          uint2 h;
          h.x = f32x2_to_bf16(g[0], g[1]);
          h.y = f32x2_to_bf16(g[2], g[3]);
          *reinterpret_cast<uint2 *>(dZ16 + e) = h;
        }
      }
    } else {
      for (int64_t r = r0 + rg; r < r1; r += RG) {
        const int64_t e = r * C + c0 + cg;
        float g = dY[e];
        if (relu && !(load_as_f32(Y, e) > 0.0f)) g = 0.0f;
        if (dZ32) dZ32[e] = g;
        if (dZ16) dZ16[e] = f32_to_bf16(g);
        a[0].add(g);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) red[threadIdx.x * 4 + i] = a[i].value();
  __syncthreads();
  if (threadIdx.x < Cw) {
    const int c = threadIdx.x, g0 = c / V, comp = c % V;
    Comp t{0.0f, 0.0f};
    for (int g = 0; g < RG; ++g) t.add(red[(g * TPR + g0) * 4 + comp]);
    dbpart[(int64_t)blockIdx.x * C + c0 + c] = t.value();
  }
}

constexpr int kMaxWgradLayers = NPVS_MAX_WGRAD_LAYERS;  // layers of one batched weight-gradient launch
constexpr int kWgSlices = 16;  // slices of each offset's pair list (at most; fewer for wide layers)
constexpr int kWgBatchBlocks = 512;  // workgroups resident at once (72 KB of LDS each: two per compute unit)
constexpr size_t kWgPartBudget = size_t(8) << 20;  // bytes of float32 slice partials aimed at

// Slices per offset: 16 while the float32 partials of every slice stay within the budget (every
// layer of at most 64 x 64 channels), fewer for wider layers, at least one.
int wg_slices(int cin, int cout) {
  const size_t per = sizeof(float) * 27 * (size_t)cin * cout;
  const size_t s = kWgPartBudget / per;
  return s < 1 ? 1 : s > (size_t)kWgSlices ? kWgSlices : (int)s;
}

// FP32 path on MFMA (v_mfma_f32_16x16x4_f32), the pair index as the contraction, four pairs to a
// product: grid (S slices, K offsets, windows of 64 input channels x 64 outputs), four waves: OG
// groups of 16 OI outputs of the window times PS = 4 / OG parts of the slice (added at the end in
// order).  A wave works alone, straight from global memory: the operand layout wants
// lane l on pair l / 16, and with channels CI m + i (m = l % 16) in block i the 16 lanes of a pair
// read its row as one contiguous CI-word piece each, one load for CI blocks:
//   A (16 x 4): lane l gives X[in][c0 + CI (l%16) + i]     B (4 x 16): dZ[out][o0 + OI (l%16) + j]
//   D: entry e of lane l is dW[c0 + CI (4 (l/16) + e) + i][o0 + OI (l%16) + j]
// Rows are loaded four products (16 pairs) ahead, indices eight; loads past the end re-read the
// last pair and are masked where they are used, like a pair member of -1 (the pair lists of the
// strided layers).  The 32 pairs of a chunk are summed by the matrix cores from zero and folded
// into compensated totals while the next chunk's products run.
// 30.6 us for the 9 699-row 64 -> 64 layer, whose products take 6.9 at the card's 152 TFLOP/s.  Bound by the
// longest slice, all workgroups running at once: the centre offset pairs every site with itself, so that its
// slices are about twice the mean (606 pairs of 310), each pair's two rows a load per product of the chain.
template <int CI, int OI, int OG, bool VEC>
__global__ __launch_bounds__(256, 2) void wgrad_f32_kernel(const float *__restrict__ X, int cin,
                                                         const float *__restrict__ dZ, int cout,
                                                         const int32_t *__restrict__ rb_off,
                                                         const int32_t *__restrict__ pairs, int S,
                                                         float *__restrict__ part) {
  constexpr int CH = 8, D = 4;  // products (of four pairs) per chunk, and how far ahead rows are loaded
  const int lane = threadIdx.x & 63, g = lane >> 4, m = lane & 15;
  constexpr int PS = 4 / OG;  // parts of the slice, one wave each
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int og = wv % OG, ps = wv / OG;
  const int k = blockIdx.y, s = blockIdx.x, otiles = (cout + 63) / 64;
  const int c0 = 64 * (blockIdx.z / otiles), o0 = 64 * (blockIdx.z % otiles) + 16 * OI * og;
  const int c = c0 + CI * m, o = o0 + OI * m;  // this lane's channels c .. c + CI - 1, outputs o .. o + OI - 1
  const int64_t pk0 = rb_off[k], pk = (int64_t)rb_off[k + 1] - pk0;
  const int64_t p0 = pk0 + pk * (s * PS + ps) / (S * PS), p1 = pk0 + pk * (s * PS + ps + 1) / (S * PS);
  const int nch = (int)((p1 - p0 + 4 * CH - 1) / (4 * CH));
  Comp tot[CI][OI][4];
#pragma unroll
  for (int i = 0; i < CI; ++i)
#pragma unroll
    for (int j = 0; j < OI; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) tot[i][j][e] = Comp{0.0f, 0.0f};
  if (nch > 0) {
    struct Pair {
      int in, out;
    };
    const int np = (int)(p1 - p0);  // pairs of this slice
    const int32_t *pl = pairs + 2 * p0;
    auto load_pair = [&](int t) {  // the pair of this lane's group in product t, or the last one
      const int p = 4 * t + g;
      Pair v;
      __builtin_memcpy(&v, pl + 2 * (int64_t)(p < np ? p : np - 1), sizeof(v));
      return v;
    };
    // lanes past the channels read channel 0 and are masked (the sign bit of an index marks a row
    // that does not exist; the masks are bit tests and ors, which leave no branch around a load)
    const float *Xc = X + (c < cin ? c : 0), *Zo = dZ + (o < cout ? o : 0);
    const int xdead = c < cin ? 0 : -1, zdead = o < cout ? 0 : -1;
    uint32_t okx = 0, okz = 0;  // validity of the rows in the slots, newest in bit 0, oldest in bit D - 1
    float x[D][CI], z[D][OI];
    Pair ip[D];
    auto load_rows = [&](int t, int q) {  // product t into slot q, through the indices of the slot
      const int past = (np - 1 - (4 * t + g)) >> 31;  // -1 past the last pair
      const int xi = ip[q].in | xdead | past, zi = ip[q].out | zdead | past;
      okx = __builtin_amdgcn_alignbit(okx, ~(uint32_t)xi, 31);  // (okx << 1) | row exists
      okz = __builtin_amdgcn_alignbit(okz, ~(uint32_t)zi, 31);
      const float *sx = Xc + (int64_t)(xi > 0 ? xi : 0) * cin, *sz = Zo + (int64_t)(zi > 0 ? zi : 0) * cout;
      if constexpr (VEC) {
        __builtin_memcpy(x[q], sx, sizeof(x[q]));
        __builtin_memcpy(z[q], sz, sizeof(z[q]));
      } else {
#pragma unroll
        for (int i = 0; i < CI; ++i) x[q][i] = sx[c + i < cin ? i : 0];
#pragma unroll
        for (int j = 0; j < OI; ++j) z[q][j] = sz[o + j < cout ? j : 0];
      }
    };
    auto masked = [](float v, uint32_t mask) {
      return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) & mask);
    };
    f32x4_t acc[2][CI][OI];
#pragma unroll
    for (int i = 0; i < CI; ++i)
#pragma unroll
      for (int j = 0; j < OI; ++j) acc[1][i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // the products of one chunk into acc[cur], while acc[cur ^ 1] of the chunk before is folded in
    auto chunk = [&](int ch, auto parity) {
      constexpr int cur = decltype(parity)::value;
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        constexpr uint32_t oldest = 1u << (D - 1);
        const uint32_t mx = okx & oldest ? ~0u : 0u, mz = okz & oldest ? ~0u : 0u;
        const int sl = q % D;
#pragma unroll
        for (int i = 0; i < CI; ++i) {
          const float av = masked(x[sl][i], VEC || c + i < cin ? mx : 0u);
#pragma unroll
          for (int j = 0; j < OI; ++j) {
            const float bv = masked(z[sl][j], VEC || o + j < cout ? mz : 0u);
            const f32x4_t from = q == 0 ? f32x4_t{0.0f, 0.0f, 0.0f, 0.0f} : acc[cur][i][j];
            acc[cur][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, from, 0, 0, 0);
          }
        }
        load_rows(ch * CH + q + D, sl);
        ip[sl] = load_pair(ch * CH + q + 2 * D);
#pragma unroll
        for (int f = q; f < CI * OI * 4; f += CH)
          tot[f / (OI * 4)][f / 4 % OI][f % 4].add(acc[cur ^ 1][f / (OI * 4)][f / 4 % OI][f % 4]);
      }
    };
#pragma unroll
    for (int q = 0; q < D; ++q) ip[q] = load_pair(q);
#pragma unroll
    for (int q = 0; q < D; ++q) {
      load_rows(q, q);
      ip[q] = load_pair(D + q);
    }
    auto fold = [&](const f32x4_t (&a)[CI][OI]) {
#pragma unroll
      for (int i = 0; i < CI; ++i)
#pragma unroll
        for (int j = 0; j < OI; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) tot[i][j][e].add(a[i][j][e]);
    };
    for (int ch = 1; ch < nch; ch += 2) {
      chunk(ch - 1, std::integral_constant<int, 0>{});
      chunk(ch, std::integral_constant<int, 1>{});
    }
    if (nch & 1) {
      chunk(nch - 1, std::integral_constant<int, 0>{});
      fold(acc[0]);
    } else {
      fold(acc[1]);
    }
  }
  // the parts of the slice, added in order into the first one's totals
  __shared__ Comp sum[PS - 1][OG][CI * OI * 4][64];
  if (ps > 0)
#pragma unroll
    for (int f = 0; f < CI * OI * 4; ++f) sum[ps - 1][og][f][lane] = tot[f / (OI * 4)][f / 4 % OI][f % 4];
  __syncthreads();
  if (ps > 0 || o0 >= cout) return;
#pragma unroll
  for (int f = 0; f < CI * OI * 4; ++f)
#pragma unroll
    for (int t = 0; t < PS - 1; ++t) tot[f / (OI * 4)][f / 4 % OI][f % 4].merge(sum[t][og][f][lane]);
#pragma unroll
  for (int i = 0; i < CI; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int ce = c0 + CI * (4 * g + e) + i;
      if (ce >= cin) continue;
      float *dst = part + ((int64_t)(k * S + s) * cin + ce) * cout + o;
#pragma unroll
      for (int j = 0; j < OI; ++j)
        if (o + j < cout) dst[j] = tot[i][j][e].value();
    }
}

template <int CI, int OI, int OG>
static void launch_wgrad_f32(const float *X, int cin, const float *dZ, int cout, int K, const int32_t *rb_off,
                             const int32_t *pairs, int S, float *part, hipStream_t s) {
  const bool vec = cin % CI == 0 && cout % OI == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
  const dim3 grid(S, K, ((cin + 63) / 64) * ((cout + 63) / 64));
  if (vec)
    wgrad_f32_kernel<CI, OI, OG, true><<<grid, 256, 0, s>>>(X, cin, dZ, cout, rb_off, pairs, S, part);
  else
    wgrad_f32_kernel<CI, OI, OG, false><<<grid, 256, 0, s>>>(X, cin, dZ, cout, rb_off, pairs, S, part);
}

// BF16 path on MFMA.  256 threads = 4 waves; a workgroup computes the window of at most 64 x 64
// entries (input channels c0 .., outputs o0 ..) that its window index selects (one window when
// cin, cout <= 64), over the pairs of its slice (sliced form, grid (S, K, windows)) or of its
// range of the whole pair list (balanced form, see wgrad_bf16_kernel).
// dW_k[c][o] = sum_p X[in_p][c] dZ[out_p][o] is a [cin x P] x [P x cout] product with the pair
// index as the contraction.  128 pairs at a time are staged into LDS transposed (channel-major,
// XT[c][p], GT[o][p]) so that both MFMA operands of v_mfma_f32_32x32x16_bf16 are one 16-byte
// LDS read per lane; wave w computes the 32 x 32 block (mb, nb) = (w / OB, w % OB):
//   A (32 x 16): lane l gives XT[mb*32 + l%32][kk + 8(l/32) + j]
//   B (16 x 32): lane l gives GT[nb*32 + l%32][kk + 8(l/32) + j]
//   D: entry r of lane l is dW[mb*32 + 8(r/4) + 4(l/32) + r%4][nb*32 + l%32]
// A staging task is 4 consecutive pairs x 8 channels of X or dZ (at most 2 per thread; the 8
// tasks of one pair quad sit in adjacent lanes).  The pair
// indices are fetched two chunks ahead and the rows of the next chunk are loaded while the
// current chunk's products run, then stored into the other LDS buffer.  Each chunk's product
// starts from zero and is added into a compensated total.
constexpr int kWgChunk = 128;
constexpr int kMaxWgOffsets = 27;  // offsets of one pair list (27 for 3^3 layers, 8 for strided ones)
constexpr int kWgPitch = kWgChunk + 16;  // bf16 elements per LDS row (padding spreads banks)
constexpr int kWgQuads = kWgChunk / 4;

// LDS position of pair p of staged row `row` (a channel): the 16-byte blocks of 8 pairs are
// permuted within the row by XOR with (row / 8) % 8 and with bit 2 of the row.  The row pitch
// (72 dwords) puts row r on 16-byte bank group (2 r + block) % 8.  A staging store writes 4 pairs
// of rows 8 cc + j for 8 channel groups cc at once: without the swizzle all 8 on one bank group,
// with it (row / 8 differs) on 8 different ones.  An MFMA operand read has 8 lanes read rows
// 8 g .. 8 g + 7 at one block: 2 r alone puts rows i and i + 4 on the same group, and bit 2
// separates them.  A block stays 16 bytes and aligned, so an operand is one 16-byte read.
__device__ __forceinline__ int wg_lds_pos(int row, int p) {
  return row * kWgPitch + ((((p >> 3) ^ (row >> 3) ^ ((row >> 2) & 1)) & 15) << 3) + (p & 7);
}

struct WgTask {
  int pq, cc;  // pair quad, 8-channel group within X (isx) or dZ
  bool isx, valid;
};

// Loads are unconditional (a missing pair reads pair pb, a missing row reads row 0; both exist
// whenever the chunk does) so that the wait before a chunk's use only covers that chunk's loads.
__device__ __forceinline__ void wg_indices(const int32_t *__restrict__ pairs, int64_t pb, int m, const WgTask &t,
                                           int *r) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = 4 * t.pq + i;
    const bool ok = t.valid && p < m;
    const int v = pairs[2 * (pb + (ok ? p : 0)) + (t.isx ? 0 : 1)];
    r[i] = ok ? v : -1;
  }
}

__device__ __forceinline__ void wg_gather(const uint16_t *__restrict__ X, int cin, const uint16_t *__restrict__ G,
                                          int cout, const WgTask &t, const int *r, uint4 *v) {
  const uint16_t *src = t.isx ? X : G;
  const int C = t.isx ? cin : cout;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool ok = r[i] >= 0;
    const uint4 x = *reinterpret_cast<const uint4 *>(src + (ok ? (int64_t)r[i] * C + 8 * t.cc : 0));
    const uint32_t m = ok ? ~0u : 0u;  // a mask, not a select of the loaded value: no branch around the load
    v[i] = make_uint4(x.x & m, x.y & m, x.z & m, x.w & m);
  }
}

__device__ __forceinline__ uint32_t word_of(const uint4 &v, int w) {
  return w == 0 ? v.x : w == 1 ? v.y : w == 2 ? v.z : v.w;
}

// Channel j of the 4 staged rows as two packed dwords (rows 0,1 and rows 2,3): one byte permute
// per dword picks the same 16-bit half of two source words (0x05040100: low halves, 0x07060302:
// high halves).
__device__ __forceinline__ void wg_store(uint16_t *XT, uint16_t *GT, const WgTask &t, const uint4 *v) {
  if (!t.valid) return;
  uint16_t *dst = t.isx ? XT : GT;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
    const uint2 pk2 = make_uint2(__builtin_amdgcn_perm(word_of(v[1], j >> 1), word_of(v[0], j >> 1), sel),
                                 __builtin_amdgcn_perm(word_of(v[3], j >> 1), word_of(v[2], j >> 1), sel));
    *reinterpret_cast<uint2 *>(dst + wg_lds_pos(8 * t.cc + j, 4 * t.pq)) = pk2;
  }
}

// The layers of one weight-gradient launch (one rulebook): layer i owns the windows
// blockIdx.z in [z0, next layer's z0).
struct WgLayer {
  const uint16_t *X, *dZ;
  float *part;
  int cin, cout, z0;
};
struct WgBatch {
  int n;
  WgLayer L[kMaxWgradLayers];
};

// A chunk: pairs [pb, pb + m) of offset k; `last` when it ends the workgroup's part of offset k
// (the partial sum of that offset is then written out).
struct WgChunk {
  int pb, m, k;
  bool last;
};

// Sliced form (G = 0): grid (S, K, windows); workgroup (s, k) takes slice s of offset k's pairs
// and writes partial slot k S + s.  Balanced form (G > 0): grid (G, 1, windows); with P pairs in
// the whole list of the K offsets and L = ceil(P / G), workgroup g takes pairs [g L, (g + 1) L)
// (clipped to P), so every workgroup has the same number of pairs whatever their spread over
// the offsets, and writes the partial of each offset k its range meets to slot g + k.  The pair
// list is ordered by offset, so a later workgroup only meets the same or later offsets: no two
// (g, k) written share a slot, and the slots number at most G + K - 1.  The workgroups that
// meet offset k (pairs [a, b)) are g = a / L .. (b - 1) / L, which is how the reduction finds
// them.
__global__ __launch_bounds__(256) void wgrad_bf16_kernel(const WgBatch B, const int32_t *__restrict__ rb_off,
                                                          const int32_t *__restrict__ pairs, int G, int K) {
  // two staging buffers: chunk ch is read from buffer ch & 1 while chunk ch + 1 is written to the
  // other one, so one barrier per chunk orders both
  __shared__ __attribute__((aligned(16))) uint16_t XT[2][64 * kWgPitch];
  __shared__ __attribute__((aligned(16))) uint16_t GT[2][64 * kWgPitch];
  __shared__ int offs[kMaxWgOffsets + 1];
  int li = 0;
  for (int i = 1; i < B.n; ++i) li = (int)blockIdx.z >= B.L[i].z0 ? i : li;
  const uint16_t *__restrict__ X = B.L[li].X;
  const uint16_t *__restrict__ dZ16 = B.L[li].dZ;
  float *__restrict__ part = B.L[li].part;
  const int cin = B.L[li].cin, cout = B.L[li].cout, z = (int)blockIdx.z - B.L[li].z0;
  const int s = blockIdx.x, S = gridDim.x, tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform (scalar)
  const int otiles = (cout + 63) / 64;
  const int c0 = 64 * (z / otiles), o0 = 64 * (z % otiles);
  const int cw = cin - c0 < 64 ? cin - c0 : 64, ow = cout - o0 < 64 ? cout - o0 : 64;  // window size
  if (tid <= K) offs[tid] = rb_off[tid];
  __syncthreads();
  // this workgroup's pairs [pA, pB) and the offset of its first pair
  int pA, pB, k0;
  if (G > 0) {
    const int64_t P = offs[K] - offs[0], L = (P + G - 1) / G;
    const int64_t a = (int64_t)s * L, b = a + L;
    pA = offs[0] + (int)(a < P ? a : P);
    pB = offs[0] + (int)(b < P ? b : P);
    k0 = 0;
    while (k0 + 1 < K && offs[k0 + 1] <= pA) ++k0;
  } else {
    k0 = blockIdx.y;
    const int64_t pk = offs[k0 + 1] - offs[k0];
    pA = offs[k0] + (int)(pk * s / S);
    pB = offs[k0] + (int)(pk * (s + 1) / S);
  }
  // chunks in order: at most kWgChunk pairs, never across an offset boundary
  auto next_chunk = [&](int &p, int &k) {
    const int end = pB < offs[k + 1] ? pB : offs[k + 1];
    const int m = end - p < kWgChunk ? end - p : kWgChunk;
    const WgChunk c{p, m, k, p + m == end};
    p += m;
    if (c.last)
      while (k + 1 < K && offs[k + 1] <= p) ++k;  // past the end of offset k (and empty offsets)
    return c;
  };
  int nch = 0;
  {
    int p = pA, k = k0;
    while (p < pB) {
      next_chunk(p, k);
      ++nch;
    }
  }
  // 32 x 32 blocks of the window: wave wv computes block (wv / OB, wv % OB) when wv < nblk
  const int CB = (cw + 31) / 32, OB = (ow + 31) / 32, nblk = CB * OB;
  const int cin8 = (cw + 7) / 8, cout8 = (ow + 7) / 8;
  // rows are read from the window's first channel on; the row pitch stays cin / cout
  const uint16_t *Xw = X + c0, *Gw = dZ16 + o0;
  // tasks of X first, then of dZ; the channel group runs fastest, so the lanes of one load
  // instruction cover whole 128-byte rows (8 lanes per row) instead of 16 bytes of 64 rows
  WgTask task[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int t = tid + 256 * u, nx = cin8 * kWgQuads;
    task[u].isx = t < nx;
    const int tt = task[u].isx ? t : t - nx, c8 = task[u].isx ? cin8 : cout8;
    task[u].cc = tt % c8;
    task[u].pq = tt / c8;
    task[u].valid = t < (cin8 + cout8) * kWgQuads;
  }
  // channel rows past cin / cout (up to the 16-row MFMA block) stay zero; the others are written
  // by every chunk
  for (int e = cw * kWgPitch / 2 + tid; e < CB * 32 * kWgPitch / 2; e += 256) {
    reinterpret_cast<uint32_t *>(XT[0])[e] = 0;
    reinterpret_cast<uint32_t *>(XT[1])[e] = 0;
  }
  for (int e = ow * kWgPitch / 2 + tid; e < OB * 32 * kWgPitch / 2; e += 256) {
    reinterpret_cast<uint32_t *>(GT[0])[e] = 0;
    reinterpret_cast<uint32_t *>(GT[1])[e] = 0;
  }
  Comp tot[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) tot[r] = Comp{0.0f, 0.0f};
  // the partial of offset k goes to slot k S + s (sliced) or s + k (balanced, s = g); entry r of
  // lane l is dW[mb 32 + 8 (r / 4) + 4 (l / 32) + r % 4][nb 32 + l % 32]
  auto write_partial = [&](int k, const Comp(&t)[16], bool zero) {
    const int64_t slot = G > 0 ? (int64_t)s + k : (int64_t)k * S + s;
    if (wv < nblk) {
      const int mb = wv / OB, nb = wv % OB;
      const int o = nb * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = mb * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (c < cw && o < ow) part[(slot * cin + c0 + c) * cout + o0 + o] = zero ? 0.0f : t[r].value();
      }
    }
  };
  // an empty slice of the sliced form still writes its (zero) slot, which the reduction reads;
  // the balanced form's reduction reads only the slots of ranges that meet an offset
  if (nch == 0) {
    if (G == 0) write_partial(k0, tot, true);
    return;
  }
  // chunk descriptors: q0 = chunk ch, q1 = ch + 1, q2 = ch + 2; the prefetches past the last
  // chunk re-read the last chunk (no branch around a load)
  int gp = pA, gk = k0;
  WgChunk q0 = next_chunk(gp, gk);
  WgChunk q1 = nch > 1 ? next_chunk(gp, gk) : q0;
  WgChunk q2 = nch > 2 ? next_chunk(gp, gk) : q1;
  int rn[2][4];
  {
    uint4 v[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      wg_indices(pairs, q0.pb, q0.m, task[u], rn[u]);
      wg_gather(Xw, cin, Gw, cout, task[u], rn[u], v[u]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      wg_indices(pairs, q1.pb, q1.m, task[u], rn[u]);
      wg_store(XT[0], GT[0], task[u], v[u]);
    }
  }
  __syncthreads();
  for (int ch = 0; ch < nch; ++ch) {
    const int cur = ch & 1;
    uint4 v[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) wg_gather(Xw, cin, Gw, cout, task[u], rn[u], v[u]);  // chunk ch + 1
#pragma unroll
    for (int u = 0; u < 2; ++u) wg_indices(pairs, q2.pb, q2.m, task[u], rn[u]);
    f32x16_t acc = {};
    {
      // a wave past nblk computes on in-range rows and is discarded at the store, so the
      // products need no branch
      const int mb = wv / OB < 1 ? wv / OB : 1, nb = wv % OB;
#pragma unroll
      for (int kk = 0; kk < kWgChunk; kk += 16) {
        const bf16x8_t a =
            *reinterpret_cast<const bf16x8_t *>(XT[cur] + wg_lds_pos(mb * 32 + (lane & 31), kk + 8 * (lane >> 5)));
        const bf16x8_t b =
            *reinterpret_cast<const bf16x8_t *>(GT[cur] + wg_lds_pos(nb * 32 + (lane & 31), kk + 8 * (lane >> 5)));
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) tot[r].add(acc[r]);
    if (q0.last) {  // the end of this workgroup's part of offset q0.k
      write_partial(q0.k, tot, false);
#pragma unroll
      for (int r = 0; r < 16; ++r) tot[r] = Comp{0.0f, 0.0f};
    }
    q0 = q1;
    q1 = q2;
    if (ch + 3 < nch) q2 = next_chunk(gp, gk);
    // the other buffer was last read in chunk ch - 1, before the barrier that ended it
#pragma unroll
    for (int u = 0; u < 2; ++u) wg_store(XT[cur ^ 1], GT[cur ^ 1], task[u], v[u]);
    __syncthreads();
  }
}

// The final reductions of the layers of one launch: layer i owns the blocks [b0, next layer's b0):
// nbw blocks for dW, then one per 4 bias channels.
struct RdLayer {
  const float *wpart, *dbpart;
  float *dW, *db;
  int cin, cout, nbw, b0, S;  // S: slices per offset of this layer's partials (sliced form)
};
struct RdBatch {
  int n;
  RdLayer L[kMaxWgradLayers];
};

// Per layer: blocks [0, nbw) reduce dW (K offsets) over the slices (grid-stride, one entry per
// thread); each block after them reduces db over the nparts partial rows for 4 channels, one wave
// per channel: lane l adds partials l, l + 64, ..., then a fixed butterfly adds the 64 lane totals;
// lane 0 writes.  G > 0: the partials are those of the balanced weight-gradient form with G
// workgroups per window over the pair list rb_off (see wgrad_bf16_kernel), added in the order of g.
__global__ __launch_bounds__(256) void grad_reduce_kernel(const RdBatch B, int nparts, int K, int G,
                                                           const int32_t *__restrict__ rb_off) {
  int li = 0;
  for (int i = 1; i < B.n; ++i) li = (int)blockIdx.x >= B.L[i].b0 ? i : li;
  const float *__restrict__ wpart = B.L[li].wpart;
  const float *__restrict__ dbpart = B.L[li].dbpart;
  float *__restrict__ dW = B.L[li].dW;
  float *__restrict__ db = B.L[li].db;
  const int cin = B.L[li].cin, cout = B.L[li].cout, nbw = B.L[li].nbw, S = B.L[li].S;
  const int bx = (int)blockIdx.x - B.L[li].b0;
  if (bx < nbw && G > 0) {  // nbw = K blocks_per_offset: block bx reduces 256 entries of one offset
    const int64_t E = (int64_t)cin * cout;
    const int per_k = (int)((E + 255) / 256), k = bx / per_k;
    const int64_t ce = (int64_t)(bx - k * per_k) * 256 + threadIdx.x;
    const int off0 = rb_off[0];
    const int64_t P = rb_off[K] - off0;
    const int a = rb_off[k] - off0, b = rb_off[k + 1] - off0;
    Comp t{0.0f, 0.0f};
    if (a < b && ce < E) {
      const uint32_t L = (uint32_t)((P + G - 1) / G);
      const int g0 = (int)((uint32_t)a / L), g1 = (int)((uint32_t)(b - 1) / L);
      const float *src = wpart + (int64_t)k * E + ce;  // slot g + k of this entry: src[g E]
      for (int g = g0; g <= g1; g += 4) {  // four slots loaded before any is added, in order of g
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = g + i <= g1 ? src[(int64_t)(g + i) * E] : 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (g + i <= g1) t.add(v[i]);
      }
    }
    if (ce < E) dW[(int64_t)k * E + ce] = t.value();
    return;
  }
  if (bx < nbw) {
    const int64_t E = (int64_t)cin * cout;
    for (int64_t e = (int64_t)bx * blockDim.x + threadIdx.x; e < K * E; e += (int64_t)nbw * blockDim.x) {
      Comp a{0.0f, 0.0f};
      const int64_t k = e / E, ce = e % E;
      if (S == kWgSlices) {  // the usual count, unrolled so that the loads are issued together
#pragma unroll
        for (int s = 0; s < kWgSlices; ++s) a.add(wpart[(k * kWgSlices + s) * E + ce]);
      } else {
        for (int s = 0; s < S; ++s) a.add(wpart[(k * S + s) * E + ce]);
      }
      dW[e] = a.value();
    }
    return;
  }
  const int o = (bx - nbw) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (o >= cout) return;  // whole waves leave together
  Comp a{0.0f, 0.0f};
  for (int s = lane; s < nparts; s += 64) a.add(dbpart[s * cout + o]);
  float t = a.value();
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
  if (lane == 0) db[o] = t;
}

npvs_status bwd_form_dz(int32_t dtype, const void *Y, const float *dY, const npvs_counts *counts, int32_t C,
                        int32_t relu, float *dZ32, uint16_t *dZ16, float *dbpart, hipStream_t s) {
  const int vec = C % 4 == 0 && (reinterpret_cast<uintptr_t>(dY) & 15) == 0 &&
                  (!relu || (reinterpret_cast<uintptr_t>(Y) & (dtype == NPVS_F32 ? 15 : 7)) == 0);
  const dim3 gz(kDbBlocks, (C + 63) / 64);
  if (dtype == NPVS_F32)
    relu_grad_kernel<float><<<gz, 256, 0, s>>>((const float *)Y, dY, counts, C, relu, vec, dZ32, nullptr, dbpart);
  else
    relu_grad_kernel<uint16_t><<<gz, 256, 0, s>>>((const uint16_t *)Y, dY, counts, C, relu, vec, nullptr, dZ16,
                                                   dbpart);
  return check_hip(hipGetLastError(), "backward: dZ");
}

npvs_status bwd_wgrad(int32_t dtype, const void *X, int32_t cin, const void *dZ, int32_t cout, int32_t K,
                      const int32_t *rb_off, const int32_t *pairs, int S, float *wpart, hipStream_t s) {
  if (dtype == NPVS_F32) {
    // blocks of 16 channels per load: as many as the (at most 64 x 64) window has, so that narrow
    // layers do not multiply by padding
    const float *x = static_cast<const float *>(X), *z = static_cast<const float *>(dZ);
#define NPVS_WG_F32(CI, OI, OG) launch_wgrad_f32<CI, OI, OG>(x, cin, z, cout, K, rb_off, pairs, S, wpart, s)
    if (cout <= 16) {
      if (cin <= 16) NPVS_WG_F32(1, 1, 1);
      else if (cin <= 32) NPVS_WG_F32(2, 1, 1);
      else NPVS_WG_F32(4, 1, 1);
    } else if (cout <= 32) {
      if (cin <= 16) NPVS_WG_F32(1, 2, 1);
      else if (cin <= 32) NPVS_WG_F32(2, 2, 1);
      else NPVS_WG_F32(4, 2, 1);
    } else {
      if (cin <= 16) NPVS_WG_F32(1, 2, 2);
      else if (cin <= 32) NPVS_WG_F32(2, 2, 2);
      else NPVS_WG_F32(4, 2, 2);
    }
#undef NPVS_WG_F32
  } else {
    WgBatch B{};
    B.n = 1;
    B.L[0] = WgLayer{(const uint16_t *)X, (const uint16_t *)dZ, wpart, cin, cout, 0};
    wgrad_bf16_kernel<<<dim3(S, K, ((cin + 63) / 64) * ((cout + 63) / 64)), 256, 0, s>>>(B, rb_off, pairs, 0, K);
  }
  return check_hip(hipGetLastError(), "backward: weight gradient");
}

static int reduce_blocks(int32_t K, int32_t cin, int32_t cout) {
  return stride_grid((int64_t)K * cin * cout, 256, 2048);
}

npvs_status bwd_reduce(const float *wpart, const float *dbpart, int nparts, int32_t K, int S, int32_t cin,
                       int32_t cout, float *dW, float *db, hipStream_t s) {
  const int nbw = reduce_blocks(K, cin, cout);
  RdBatch B{};
  B.n = 1;
  B.L[0] = RdLayer{wpart, dbpart, dW, db, cin, cout, nbw, 0, S};
  grad_reduce_kernel<<<nbw + (cout + 3) / 4, 256, 0, s>>>(B, nparts, K, 0, nullptr);
  return check_hip(hipGetLastError(), "backward: reductions");
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace: float32 dZ (FP32 path), bfloat16 dZ (BF16 path), the slice partials of dW, the bias
// partials, and the split-input partials of the data gradient (BF16 layers with 1024+ outputs,
// whose data gradient reads that many channels).
static void bwd_ws_layout(int32_t cin, int32_t cout, int32_t cap, int32_t dtype, size_t *o_dz32, size_t *o_dz16,
                          size_t *o_wp, size_t *o_dbp, size_t *o_dx, size_t *dx_bytes, size_t *bytes) {
  size_t o = 0;
  *o_dz32 = o;
  if (dtype == NPVS_F32) o += align256(sizeof(float) * (size_t)cap * cout);
  *o_dz16 = o;
  if (dtype == NPVS_BF16) o += align256(sizeof(uint16_t) * (size_t)cap * cout);
  *o_wp = o;
  o += align256(sizeof(float) * 27 * wg_slices(cin, cout) * (size_t)cin * cout);
  *o_dbp = o;
  o += align256(sizeof(float) * kDbBlocks * (size_t)cout);
  *o_dx = o;
  *dx_bytes = conv_fwd_ws_bytes(cout, cin, cap, dtype);
  o += align256(*dx_bytes);
  *bytes = o;
}

void bwd_ws_dz_parts(int32_t cin, int32_t cout, int32_t cap, size_t *o_dz16, size_t *o_dbpart, size_t *bytes) {
  size_t a, c, e, f;
  bwd_ws_layout(cin, cout, cap, NPVS_BF16, &a, o_dz16, &c, o_dbpart, &e, &f, bytes);
}

}  // namespace npvs

using namespace npvs;

extern "C" npvs_status npvs_conv_bwd_workspace_size(int32_t cin, int32_t cout, int32_t cap_sites, int32_t dtype,
                                                    size_t *bytes) {
  if (!bytes || cin < 1 || cout < 1 || cap_sites < 1)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_conv_bwd_workspace_size: bad arguments");
  size_t a, b, c, d, e, f;
  bwd_ws_layout(cin, cout, cap_sites, dtype, &a, &b, &c, &d, &e, &f, bytes);
  return NPVS_OK;
}

// One event per thread and device orders a second stream after the first.  Re-recording it is
// safe: a wait takes the state the event had when the wait was enqueued.
static npvs_status fork_event(hipEvent_t *ev) {
  constexpr int kMaxDevices = 64;
  thread_local hipEvent_t events[kMaxDevices] = {};
  int dev = 0;
  npvs_status st = check_hip(hipGetDevice(&dev), "backward stream join");
  if (st != NPVS_OK) return st;
  if (dev < 0 || dev >= kMaxDevices) return fail(NPVS_ERR_UNSUPPORTED, "backward stream join: device index");
  if (!events[dev]) {
    st = check_hip(hipEventCreateWithFlags(&events[dev], hipEventDisableTiming), "backward stream join");
    if (st != NPVS_OK) return st;
  }
  *ev = events[dev];
  return NPVS_OK;
}

// s2 waits for the work enqueued so far on s (no-op when they are the same stream).
static npvs_status join_after(hipStream_t s, hipStream_t s2) {
  if (s2 == s) return NPVS_OK;
  hipEvent_t ev;
  npvs_status st = fork_event(&ev);
  if (st == NPVS_OK) st = check_hip(hipEventRecord(ev, s), "backward stream join");
  if (st == NPVS_OK) st = check_hip(hipStreamWaitEvent(s2, ev, 0), "backward stream join");
  return st;
}

// dZ and the bias partials on s; the data gradient on s; the weight gradient on s2 and the
// reductions on s3 (s2 first waits for the dZ of s, s3 for the weight gradient of s2; equal
// streams need no wait).
static npvs_status conv_bwd(const void *X, int32_t cin, const void *Wt, int32_t cout, const void *Y, const float *dY,
                            const int32_t *nbr, const int32_t *rb_off, const int32_t *rb_pairs,
                            const npvs_counts *counts, int32_t cap_sites, int32_t dtype, int32_t relu, float *dX,
                            float *dW, float *db, void *ws, size_t ws_bytes, hipStream_t s, hipStream_t s2,
                            hipStream_t s3) {
  if (!X || !dY || !nbr || !rb_off || !rb_pairs || !counts || !ws || (relu && !Y) || (dX && !Wt))
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_bwd: null pointer");
  if (!dW != !db) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_bwd: dW and db must both be given or both null");
  if (cin < 1 || cout < 1 || cap_sites < 1) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_bwd: bad sizes");
  if (dtype != NPVS_F32 && dtype != NPVS_BF16)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_bwd: dtype must be NPVS_F32 or NPVS_BF16");
  if (dtype == NPVS_BF16 && (cin % 8 || cout % 8))
    return fail(NPVS_ERR_UNSUPPORTED, "npvs_sparse_conv_bwd: BF16 needs cin % 8 == 0 and cout % 8 == 0");
  size_t o32, o16, owp, odb, odx, dx_bytes, need;
  bwd_ws_layout(cin, cout, cap_sites, dtype, &o32, &o16, &owp, &odb, &odx, &dx_bytes, &need);
  if (ws_bytes < need) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_bwd: workspace too small");
  char *w = static_cast<char *>(ws);
  // the FP32 path keeps dZ in float32, the BF16 path in bfloat16 only (both of its products read it)
  float *dZ32 = dtype == NPVS_F32 ? reinterpret_cast<float *>(w + o32) : nullptr;
  uint16_t *dZ16 = dtype == NPVS_BF16 ? reinterpret_cast<uint16_t *>(w + o16) : nullptr;
  float *wpart = reinterpret_cast<float *>(w + owp);
  float *dbpart = reinterpret_cast<float *>(w + odb);
  npvs_status st = bwd_form_dz(dtype, Y, dY, counts, cout, relu, dZ32, dZ16, dbpart, s);
  if (st != NPVS_OK) return st;
  if (dW) st = join_after(s, s2);
  if (st != NPVS_OK) return st;
  if (dX) {
    st = conv_fwd_dispatch(dtype == NPVS_F32 ? (const void *)dZ32 : (const void *)dZ16, cout, Wt, nullptr, cin, nbr,
                           counts, cap_sites, dtype, 0, 1, dX, s, kDefaultConvVariant, dx_bytes ? w + odx : nullptr,
                           dx_bytes);
    if (st != NPVS_OK) return st;
  }
  if (!dW) return NPVS_OK;  // dZ and the bias partials stay in ws for npvs_sparse_conv_wgrad
  const int S = wg_slices(cin, cout);
  st = bwd_wgrad(dtype, X, cin, dtype == NPVS_F32 ? (const void *)dZ32 : (const void *)dZ16, cout, 27, rb_off,
                 rb_pairs, S, wpart, s2);
  if (st == NPVS_OK) st = join_after(s2, s3);
  if (st != NPVS_OK) return st;
  return bwd_reduce(wpart, dbpart, kDbBlocks, 27, S, cin, cout, dW, db, s3);
}


extern "C" npvs_status npvs_sparse_conv_bwd(const void *X, int32_t cin, const void *Wt, int32_t cout, const void *Y,
                                           const float *dY, const int32_t *nbr, const int32_t *rb_off,
                                           const int32_t *rb_pairs, const npvs_counts *counts, int32_t cap_sites,
                                           int32_t dtype, int32_t relu, float *dX, float *dW, float *db, void *ws,
                                           size_t ws_bytes, void *stream, void *wgrad_stream, void *reduce_stream) {
  const hipStream_t s = as_stream(stream);
  const hipStream_t s2 = wgrad_stream ? as_stream(wgrad_stream) : s;
  const hipStream_t s3 = reduce_stream ? as_stream(reduce_stream) : s2;
  return conv_bwd(X, cin, Wt, cout, Y, dY, nbr, rb_off, rb_pairs, counts, cap_sites, dtype, relu, dX, dW, db, ws,
                  ws_bytes, s, s2, s3);
}

extern "C" npvs_status npvs_sparse_conv_wgrad(int32_t n_layers, const npvs_wgrad_layer *layers,
                                             const int32_t *rb_off, const int32_t *rb_pairs, int32_t cap_sites,
                                             int32_t dtype, int32_t slices, void *stream) {
  if (!layers || !rb_off || !rb_pairs) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_wgrad: null pointer");
  if (n_layers < 1 || n_layers > NPVS_MAX_WGRAD_LAYERS || cap_sites < 1 || slices < 0)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_wgrad: bad sizes");
  if (dtype != NPVS_F32 && dtype != NPVS_BF16)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_wgrad: dtype must be NPVS_F32 or NPVS_BF16");
  int S = kWgSlices, windows = 0;
  for (int i = 0; i < n_layers; ++i) {
    const npvs_wgrad_layer &l = layers[i];
    if (!l.X || !l.ws || !l.dW || !l.db) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_wgrad: null pointer");
    if (l.cin < 1 || l.cout < 1) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_wgrad: bad sizes");
    if (dtype == NPVS_BF16 && (l.cin % 8 || l.cout % 8))
      return fail(NPVS_ERR_UNSUPPORTED, "npvs_sparse_conv_wgrad: BF16 needs cin % 8 == 0 and cout % 8 == 0");
    size_t a, b, c, d, e, f, need;
    bwd_ws_layout(l.cin, l.cout, cap_sites, dtype, &a, &b, &c, &d, &e, &f, &need);
    if (l.ws_bytes < need) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_wgrad: workspace too small");
    const int sl = wg_slices(l.cin, l.cout);
    S = sl < S ? sl : S;
    windows += ((l.cin + 63) / 64) * ((l.cout + 63) / 64);
  }
  // BF16 with slices = 0: the balanced form, at most kWgBatchBlocks workgroups in all so that they
  // run in one round, and at most as many per window as the partial slots allow (G + 26 slots of
  // the 27 S the workspace holds); otherwise the sliced form with `slices` slices per offset
  int G = 0;
  if (slices > 0) {
    S = slices < S ? slices : S;
  } else if (dtype == NPVS_BF16) {
    const int want = kWgBatchBlocks / windows, cap = 27 * S - 26;
    G = want < cap ? want : cap;
    G = G < 1 ? 1 : G;
  }
  const hipStream_t s = as_stream(stream);
  WgBatch W{};
  RdBatch R{};
  W.n = R.n = n_layers;
  int z0 = 0, b0 = 0;
  for (int i = 0; i < n_layers; ++i) {
    const npvs_wgrad_layer &l = layers[i];
    size_t o32, o16, owp, odb, odx, dxb, need;
    bwd_ws_layout(l.cin, l.cout, cap_sites, dtype, &o32, &o16, &owp, &odb, &odx, &dxb, &need);
    char *w = static_cast<char *>(l.ws);
    float *wpart = reinterpret_cast<float *>(w + owp);
    const float *dbpart = reinterpret_cast<const float *>(w + odb);
    // FP32: one launch per layer (the FP32 kernel's grid is per layer), each with the layer's own
    // slice count (or `slices` when smaller)
    int Sl = S;
    if (dtype == NPVS_F32) {
      Sl = wg_slices(l.cin, l.cout);
      Sl = slices > 0 && slices < Sl ? slices : Sl;
      const npvs_status st = bwd_wgrad(dtype, l.X, l.cin, w + o32, l.cout, 27, rb_off, rb_pairs, Sl, wpart, s);
      if (st != NPVS_OK) return st;
    }
    W.L[i] = WgLayer{(const uint16_t *)l.X, reinterpret_cast<const uint16_t *>(w + o16), wpart, l.cin, l.cout, z0};
    z0 += ((l.cin + 63) / 64) * ((l.cout + 63) / 64);
    const int nbw = G > 0 ? 27 * (int)(((int64_t)l.cin * l.cout + 255) / 256) : reduce_blocks(27, l.cin, l.cout);
    R.L[i] = RdLayer{wpart, dbpart, l.dW, l.db, l.cin, l.cout, nbw, b0, Sl};
    b0 += nbw + (l.cout + 3) / 4;
  }
  if (dtype == NPVS_BF16) {
    const dim3 grid = G > 0 ? dim3(G, 1, z0) : dim3(S, 27, z0);
    wgrad_bf16_kernel<<<grid, 256, 0, s>>>(W, rb_off, rb_pairs, G, 27);
    const npvs_status st = check_hip(hipGetLastError(), "npvs_sparse_conv_wgrad: weight gradient");
    if (st != NPVS_OK) return st;
  }
  grad_reduce_kernel<<<b0, 256, 0, s>>>(R, kDbBlocks, 27, G, rb_off);
  return check_hip(hipGetLastError(), "npvs_sparse_conv_wgrad: reductions");
}

extern "C" npvs_status npvs_sparse_conv_dgrad_relu(const void *Wt, int32_t cin, int32_t cout, const void *M,
                                                  int32_t cin_below, const int32_t *nbr, const npvs_counts *counts,
                                                  int32_t cap_sites, const void *ws, size_t ws_bytes,
                                                  void *ws_below, size_t ws_below_bytes, void *stream) {
  if (!Wt || !nbr || !counts || !ws || !ws_below)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_dgrad_relu: null pointer");
  if (cin < 1 || cout < 1 || cin_below < 1 || cap_sites < 1)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_dgrad_relu: bad sizes");
  if (ws == ws_below) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_dgrad_relu: ws and ws_below must differ");
  if (cin > 64 || cout > 64 || cin % 8 || cout % 8 || cin_below % 8)
    return fail(NPVS_ERR_UNSUPPORTED,
                "npvs_sparse_conv_dgrad_relu: needs cin, cout <= 64 and cin, cout, cin_below multiples of 8");
  size_t a, o16, c, d, e, f, need;
  bwd_ws_layout(cin, cout, cap_sites, NPVS_BF16, &a, &o16, &c, &d, &e, &f, &need);
  if (ws_bytes < need) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_dgrad_relu: workspace too small");
  size_t b16, bdb;
  bwd_ws_layout(cin_below, cin, cap_sites, NPVS_BF16, &a, &b16, &c, &bdb, &e, &f, &need);
  if (ws_below_bytes < need)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_dgrad_relu: workspace of the layer below too small");
  const uint16_t *dZ = reinterpret_cast<const uint16_t *>(static_cast<const char *>(ws) + o16);
  char *wb = static_cast<char *>(ws_below);
  return dgrad_relu_fused(dZ, cout, Wt, cin, nbr, counts, cap_sites, static_cast<const uint16_t *>(M),
                          reinterpret_cast<uint16_t *>(wb + b16), reinterpret_cast<float *>(wb + bdb),
                          as_stream(stream));
}
