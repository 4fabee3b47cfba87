// Submanifold sparse 3x3x3 convolution, forward (Sec. 2.3, 3.3):
//   Y[r][o] = act(b[o] + sum_k sum_c X[nbr[k][r]][c] W[k][c][o])
// Output-stationary gather-GEMM: a tile of output rows loops over the 27 offsets, gathers the
// neighbour rows of each offset and multiplies them by W_k.  Each offset really is a dense
// [rows x Cin] x [Cin x Cout] contraction, so the BF16 path runs it on MFMA.
#include <type_traits>

#include "conv_common.hpp"

namespace npvs {

// ------------------------------------------------------------------------------------------
// Weight packing.  P is the conv weight a kernel reads, [27][CI][CO]:
//   plain: P[k][c][o] = W[k][c][o]            (CI = cin,  CO = cout)
//   flip : P[k][c][o] = W[26-k][o][c]         (CI = cout, CO = cin; the data-gradient weight)
// F32 layout: P itself.  BF16 layout: MFMA A-operand fragments of P^T for
// v_mfma_f32_16x16x32_bf16, Wp[k][nb][kb][lane][j] = P[k][kb*32 + 8*(lane/16) + j][nb*16 + lane%16]
// (zero outside CI x CO), so each lane loads its 8 values with one 16-byte load.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float packed_src(const float *W, int cin, int cout, int flip, int k, int c, int o) {
  return flip ? W[((int64_t)(26 - k) * cin + o) * cout + c] : W[((int64_t)k * cin + c) * cout + o];
}

__global__ void pack_f32_kernel(const float *__restrict__ W, int cin, int cout, int flip, float *__restrict__ P) {
  const int CI = flip ? cout : cin, CO = flip ? cin : cout;
  const int64_t total = 27LL * CI * CO;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    int o = e % CO, c = (e / CO) % CI, k = e / ((int64_t)CO * CI);
    P[e] = packed_src(W, cin, cout, flip, k, c, o);
  }
}

__device__ __forceinline__ void pack_bf16_entry(const float *__restrict__ W, int cin, int cout, int flip,
                                                uint16_t *__restrict__ P, int64_t e) {
  const int CI = flip ? cout : cin, CO = flip ? cin : cout;
  const int KB = (CI + 31) / 32, NB = (CO + 15) / 16;
  int j = e & 7, lane = (e >> 3) & 63;
  int64_t f = e >> 9;  // fragment index (k, nb, kb)
  int kb = f % KB, nb = (f / KB) % NB, k = f / ((int64_t)KB * NB);
  int c = kb * 32 + 8 * (lane >> 4) + j, o = nb * 16 + (lane & 15);
  float v = (c < CI && o < CO) ? packed_src(W, cin, cout, flip, k, c, o) : 0.0f;
  P[e] = f32_to_bf16(v);
}

// The buffer holds npvs_packed_weight_bytes() bytes, sized for the larger orientation; entries
// past this orientation's fragments are zero, so the whole buffer is defined.
__global__ void pack_bf16_kernel(const float *__restrict__ W, int cin, int cout, int flip, int64_t buf_elems,
                                 uint16_t *__restrict__ P) {
  const int CI = flip ? cout : cin, CO = flip ? cin : cout;
  const int64_t total = 27LL * ((CO + 15) / 16) * ((CI + 31) / 32) * 64 * 8;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < buf_elems; e += (int64_t)gridDim.x * blockDim.x) {
    if (e < total) pack_bf16_entry(W, cin, cout, flip, P, e);
    else P[e] = 0;
  }
}

// Batched packing: blockIdx.y selects the entry; each entry is grid-strided over blockIdx.x.
struct PackBatch {
  npvs_pack_desc d[NPVS_MAX_PACK];
  int64_t elems[NPVS_MAX_PACK];  // buffer entries (npvs_packed_weight_bytes / element size)
};

__global__ void pack_batch_kernel(PackBatch PB, int dtype) {
  const npvs_pack_desc &D = PB.d[blockIdx.y];
  const int flip = D.flip_transpose ? 1 : 0;
  const int CI = flip ? D.cout : D.cin, CO = flip ? D.cin : D.cout;
  const int64_t total = dtype == NPVS_F32 ? 27LL * CI * CO : 27LL * ((CO + 15) / 16) * ((CI + 31) / 32) * 64 * 8;
  const int64_t buf = PB.elems[blockIdx.y];
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < buf; e += (int64_t)gridDim.x * blockDim.x) {
    if (e >= total) {
      static_cast<uint16_t *>(D.Wp)[e] = 0;  // only the BF16 layout has a tail
    } else if (dtype == NPVS_F32) {
      const int o = e % CO, c = (e / CO) % CI, k = e / ((int64_t)CO * CI);
      static_cast<float *>(D.Wp)[e] = packed_src(D.W, D.cin, D.cout, flip, k, c, o);
    } else {
      pack_bf16_entry(D.W, D.cin, D.cout, flip, static_cast<uint16_t *>(D.Wp), e);
    }
  }
}

// ------------------------------------------------------------------------------------------
// FP32 path on MFMA (v_mfma_f32_16x16x4_f32: float32 operands and accumulation), any channel
// counts; the order of a sum follows from the channel counts alone.  A workgroup of NW waves computes 16 MB rows x 16 NI outputs; the contraction over
// (offset, input channel) is cut into substeps of 16 channels of one offset, dealt to the waves in
// turn, so a wave's rows and weights are its own and nothing is shared (no barrier) until the NW
// partial results are added in LDS in a fixed order.  The product is computed transposed
// (D = W^T X^T).  The channels of a substep are taken in the order 4 g + j (lane group g = l / 16,
// product j) and output block i holds the outputs NI m + i, so that every load is as wide as the
// loader takes it (a load costs one cycle per 4 lanes whatever their width):
//   A (16 x 4): lane l gives W[k][16 cc + 4 g + j][NI (l%16) + i]   one NI-word load serves NI blocks
//   B (4 x 16): lane l gives X[row l%16][16 cc + 4 g + j]            one 16-byte LDS read serves 4 products
//   D: lane l holds the 4 NI consecutive outputs from 4 NI g on of row l%16
// The gathered rows go through LDS (wave-private, two buffers) because the operand layout puts
// adjacent lanes on different rows, which loads at 67 cycles a KB against 26 with four adjacent
// lanes on one row's 64 bytes.  LDS serves a wave's accesses in order, and a wave-scope fence per substep
// (no instruction) keeps the compiler to it.  Rows are loaded two substeps ahead, indices three,
// weights one.
// Bound by the matrix cores: the busiest compute unit of the 9 699-row 64 -> 64 layer has 1 296
// products of 32 cycles per SIMD, 17 us of its 32.6 (113 us with vector FMA; without any load the
// same loop takes 25), the rest being the launch and the first index, row and weight round trips.
// ------------------------------------------------------------------------------------------
// All ones when ok, as a value whose origin the compiler does not see: a mask on a loaded value
// (or on its index) then stays a mask, instead of becoming a branch around the load.
__device__ __forceinline__ uint32_t lane_mask(bool ok) {
  uint32_t m = ok ? ~0u : 0u;
  asm volatile("" : "+v"(m));
  return m;
}
__device__ __forceinline__ float and_mask(float v, uint32_t m) {
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) & m);
}

// LDS: two buffers of rows per wave (64 bytes a row), later half of the waves' partial results
// (16 MB rows of 16 NI + 4 floats, the 4 against bank conflicts)
constexpr int f32_lds_words(int MB, int NI, int NW) {
  const int rows = NW * 2 * 16 * MB * 4, part = NW / 2 * 16 * MB * (4 * NI + 1);
  return rows > part ? rows : part;  // 16-byte words
}

// How the weights and rows may be read: kF32Full: cin % 16 == 0, cout % (16 NI) == 0; kF32Vec:
// cin % 4 == 0, cout % NI == 0 (whole vectors, some of them outside); kF32Any: word by word.
enum F32Access { kF32Full, kF32Vec, kF32Any };

template <int N> struct FloatVec { float v[N]; };

template <int MB, int NI, int NW, F32Access ACC>
__device__ __forceinline__ void conv_f32_body(float4 *lds, const float *__restrict__ X, int cin,
                                              const float *__restrict__ P, const float *__restrict__ bias, int cout,
                                              const int32_t *__restrict__ nbr, int n, int cap, int relu,
                                              float *__restrict__ Y) {
  constexpr int ROWS = 16 * MB, RP = 4 * NI + 1;  // RP: 16-byte words per partial row
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, m = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform (scalar)
  const int C16 = (cin + 15) / 16, U = 27 * C16, S = (U - wv + NW - 1) / NW;  // substeps wv, wv + NW, ...
  const int kq = NW / C16, cq = NW % C16;  // the advance in (offset, 16-channel chunk) per substep of a wave
  const int ntiles = (n + ROWS - 1) / ROWS, groups = (cout + 16 * NI - 1) / (16 * NI), nunits = ntiles * groups;
  float4 *rows = lds + wv * 2 * ROWS * 4;
  // word q of row r sits at slot q ^ swz(r): the 8 (or 16) lanes of one LDS pass, on consecutive
  // rows at one q, then fall on different banks
  auto swz = [](int r) { return ((r >> 1) ^ (r >> 3)) & 3; };
  for (int j = 0;; ++j) {
    const int unit = xcd_tile(blockIdx.x, gridDim.x, nunits, j);
    if (unit < 0) break;
    const int row0 = unit / groups * ROWS, o0 = unit % groups * 16 * NI, o = o0 + NI * m;
    int k = wv / C16, cc = wv % C16;   // (offset, chunk) of the index loads
    int wk = k, wc = cc;               // and of the weight loads
    auto advance = [&](int &a, int &b) {
      a += kq;
      b += cq;
      if (b >= C16) {
        b -= C16;
        ++a;
      }
    };
    // Loads retire in order, so a value used right after its load makes every earlier load wait:
    // indices, rows and weights are loaded raw and judged where they are used.  Loads past the
    // last substep re-read valid places and are not used.
    struct Index {
      int i[MB], c;  // raw indices and the channel they are for
    };
    auto next_index = [&]() {
      Index ix;
#pragma unroll
      for (int u = 0; u < MB; ++u) {
        const int r = row0 + 16 * u + (lane >> 2);
        ix.i[u] = nbr[(int64_t)(k < 27 ? k : 26) * cap + (r < n ? r : n - 1)];
      }
      ix.c = 16 * cc + 4 * (lane & 3);
      advance(k, cc);
      return ix;
    };
    auto load_rows = [&](const Index &ix, float4 (&x)[MB], int (&left)[MB]) {  // left: how many of the channels exist
#pragma unroll
      for (int u = 0; u < MB; ++u) {
        left[u] = ix.i[u] >= 0 && row0 + 16 * u + (lane >> 2) < n ? cin - ix.c : 0;
        const float *src = X + (left[u] > 0 ? (int64_t)ix.i[u] * cin + ix.c : 0);
        if constexpr (ACC != kF32Any) {
          __builtin_memcpy(&x[u], src, sizeof(x[u]));  // one load, at any word's address
        } else {
          x[u].x = src[0];
          x[u].y = src[lane_mask(left[u] > 1) & 1u];
          x[u].z = src[lane_mask(left[u] > 2) & 2u];
          x[u].w = src[lane_mask(left[u] > 3) & 3u];
        }
      }
    };
    auto store_rows = [&](int buf, const float4 (&x)[MB], const int (&left)[MB]) {
#pragma unroll
      for (int u = 0; u < MB; ++u) {
        const int r = 16 * u + (lane >> 2);
        const uint32_t m0 = lane_mask(left[u] > 0), m1 = ACC != kF32Any ? m0 : lane_mask(left[u] > 1),
                       m2 = ACC != kF32Any ? m0 : lane_mask(left[u] > 2),
                       m3 = ACC != kF32Any ? m0 : lane_mask(left[u] > 3);
        rows[(buf * ROWS + r) * 4 + ((lane & 3) ^ swz(r))] =
            make_float4(and_mask(x[u].x, m0), and_mask(x[u].y, m1), and_mask(x[u].z, m2), and_mask(x[u].w, m3));
      }
    };
    auto load_weights = [&](float (&w)[4][NI], int &left) {  // left: of the channels from 4 g on, how many exist
      const int c = 16 * wc + 4 * g;
      left = o < cout ? cin - c : 0;
      const bool any = ACC == kF32Full || left > 0;
      const float *src = P + (any ? ((int64_t)(wk < 27 ? wk : 26) * cin + c) * cout + o : 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float *s = src + (ACC == kF32Full ? (uint32_t)(q * cout) : (uint32_t)(q * cout) & lane_mask(left > q));
        if constexpr (ACC == kF32Any || NI == 1) {
#pragma unroll
          for (int i = 0; i < NI; ++i) w[q][i] = s[i == 0 ? 0u : (uint32_t)i & lane_mask(o + i < cout)];
        } else {
          FloatVec<NI> v;
          __builtin_memcpy(&v, s, sizeof(v));
#pragma unroll
          for (int i = 0; i < NI; ++i) w[q][i] = v.v[i];
        }
      }
      advance(wk, wc);
    };
    f32x4_t acc[MB][NI];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[mb][i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float4 x[2][MB];
    float w[2][4][NI];
    int xl[2][MB], wl[2];
    const Index ix0 = next_index(), ix1 = next_index();
    Index ix = next_index();
    load_weights(w[0], wl[0]);
    load_rows(ix0, x[0], xl[0]);
    load_rows(ix1, x[1], xl[1]);
    store_rows(0, x[0], xl[0]);
    // substep s (parity cur): its rows are in LDS, those of the next in x[cur ^ 1], indices two ahead in ix
    auto step = [&](auto parity) {
      constexpr int cur = decltype(parity)::value;
      // the rows stored at the end of the step before come before this step's reads of them, and the
      // reads of the step before come before this step's store: of other lanes' words, so said here
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
      load_rows(ix, x[cur], xl[cur]);
      ix = next_index();
      load_weights(w[cur ^ 1], wl[cur ^ 1]);
      float4 b[MB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) b[mb] = rows[(cur * ROWS + mb * 16 + m) * 4 + (g ^ swz(mb * 16 + m))];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t mq = ACC == kF32Full ? 0u : lane_mask(wl[cur] > q);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float av = w[cur][q][i];
          if constexpr (ACC == kF32Vec) av = and_mask(av, mq);
          if constexpr (ACC == kF32Any) av = and_mask(av, mq & lane_mask(o + i < cout));
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const float bv = q == 0 ? b[mb].x : q == 1 ? b[mb].y : q == 2 ? b[mb].z : b[mb].w;
            acc[mb][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[mb][i], 0, 0, 0);
          }
        }
      }
      store_rows(cur ^ 1, x[cur ^ 1], xl[cur ^ 1]);
    };
    for (int s = 1; s < S; s += 2) {
      step(std::integral_constant<int, 0>{});
      step(std::integral_constant<int, 1>{});
    }
    if (S & 1) step(std::integral_constant<int, 0>{});
    // the partial results: the upper half of the waves hand theirs to the lower half, then all
    // threads add the sums of their 16-byte words in wave order
    float4 *part = lds + (wv % (NW / 2)) * ROWS * RP;
    auto word = [&](int mb, int f) {  // words f of the 4 NI consecutive outputs of this lane
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[mb][(4 * f + e) % NI][(4 * f + e) / NI];
      return make_float4(v[0], v[1], v[2], v[3]);
    };
    __syncthreads();  // every wave is done with its rows
    if (wv >= NW / 2)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int f = 0; f < NI; ++f) part[(mb * 16 + m) * RP + g * NI + f] = word(mb, f);
    __syncthreads();
    if (wv < NW / 2)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int f = 0; f < NI; ++f) {
          float4 *p = part + (mb * 16 + m) * RP + g * NI + f;
          const float4 a = word(mb, f), b = *p;
          *p = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
        }
    __syncthreads();
    for (int e = tid; e < ROWS * 4 * NI; e += 64 * NW) {
      const int rr = e / (4 * NI), f = e % (4 * NI), r = row0 + rr, oo = o0 + 4 * f;
      if (r >= n || oo >= cout) continue;
      float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < NW / 2; ++s) {
        const float4 p = lds[(s * ROWS + rr) * RP + f];
        v[0] += p.x;
        v[1] += p.y;
        v[2] += p.z;
        v[3] += p.w;
      }
      float *dst = Y + (int64_t)r * cout + oo;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (ACC != kF32Full && oo + i >= cout) break;
        const float t = v[i] + (bias ? bias[oo + i] : 0.0f);
        dst[i] = (relu && t < 0.0f) ? 0.0f : t;
      }
    }
    __syncthreads();  // before the next unit's rows
  }
}

// Rows per workgroup: 48, which read the weights a third as often as 16, when that takes no more
// rounds over the 256 compute units than 16 do, or when there are enough units (two a compute unit)
// that rounds do not matter.  64 -> 64: 9 699 rows 32.6 us (16 rows: 35.6), 94 371 rows 211 (247);
// 1 802 rows 14.8 us with 16 (48 rows: 30.5).
template <int NI, int NW, F32Access ACC>
__global__ __launch_bounds__(64 * NW, ACC == kF32Any ? 2 : 3) void conv_fwd_f32_kernel(const float *__restrict__ X, int cin,
                                                                const float *__restrict__ P,
                                                                const float *__restrict__ bias, int cout,
                                                                const int32_t *__restrict__ nbr,
                                                                const npvs_counts *__restrict__ counts, int cap,
                                                                int relu, float *__restrict__ Y) {
  __shared__ float4 lds[f32_lds_words(3, NI, NW)];
  const int32_t n = counts->n_sites;
  const int groups = (cout + 16 * NI - 1) / (16 * NI);
  const int64_t t1 = (n + 15) / 16 * (int64_t)groups, t3 = (n + 47) / 48 * (int64_t)groups;
  if (t3 >= 512 || 3 * ((t3 + 255) / 256) <= (t1 + 255) / 256)
    conv_f32_body<3, NI, NW, ACC>(lds, X, cin, P, bias, cout, nbr, n, cap, relu, Y);
  else
    conv_f32_body<1, NI, NW, ACC>(lds, X, cin, P, bias, cout, nbr, n, cap, relu, Y);
}

template <int NI>
static void launch_conv_f32(const float *X, int cin, const float *P, const float *bias, int cout, const int32_t *nbr,
                            const npvs_counts *counts, int cap, int relu, float *Y, hipStream_t s) {
  const int64_t units = (int64_t)((cap + 15) / 16) * ((cout + 16 * NI - 1) / (16 * NI));
  const int G = units > 2048 ? 2048 : (int)((units + 7) & ~7);
  // by the channel counts alone: the number of waves is the order of the sums, which X's address may not
  // change (an unaligned 16-byte load is one instruction too)
  const bool vec = cin % 4 == 0 && cout % NI == 0;
  // 4 waves (three workgroups a compute unit hide each other's start and end), or 8 from 256 input
  // channels on, where a wave's chain is long and the sites are few (512 -> 64, 1 802 rows: 80 us
  // against 104; 64 -> 64, 94 371 rows: 232 against 211)
#define NPVS_F32_LAUNCH(NW, ACC) \
  conv_fwd_f32_kernel<NI, NW, ACC><<<G, 64 * NW, 0, s>>>(X, cin, P, bias, cout, nbr, counts, cap, relu, Y)
  if (!vec) NPVS_F32_LAUNCH(4, kF32Any);
  else if (cin % 16 || cout % (16 * NI)) NPVS_F32_LAUNCH(4, kF32Vec);
  else if (cin >= 256) NPVS_F32_LAUNCH(8, kF32Full);
  else NPVS_F32_LAUNCH(4, kF32Full);
#undef NPVS_F32_LAUNCH
}

// ------------------------------------------------------------------------------------------
// BF16 path on MFMA (v_mfma_f32_16x16x32_bf16, FP32 accumulation).
// The product is computed transposed, D = W^T X^T, so that a lane's accumulator holds four
// consecutive output channels of one row (a single 8- or 16-byte store):
//   A (16 x 32) = W^T block: lane l gives W[kb*32 + 8(l/16) + j][nb*16 + l%16]   (packed, one load)
//   B (32 x 16) = X^T block: lane l gives X[row0 + l%16][kb*32 + 8(l/16) + j]    (gathered row, one load)
//   D (16 x 16): lane l holds Y[row0 + l%16][nb*16 + 4(l/16) + i], i = 0..3
// A wave owns MB x 16 rows and all NB x 16 output channels.  The KSPLIT waves of a workgroup
// take consecutive slices of 27 / KSPLIT offsets of the same rows.  A wave loads the neighbour
// indices of all its offsets at once, then loads the row and weight fragments of offset q + 1
// while the MFMAs of offset q run; offsets where none of its rows has a neighbour are skipped.
// The partial sums of the waves are added in LDS in wave order (deterministic) and every wave
// finishes some of the 16 x 16 output blocks (bias, ReLU, rounding, store).
// ------------------------------------------------------------------------------------------
// 8 channels [c, c + 8) of row i of X, or zero when i < 0 or c >= cin.  The load itself is
// unconditional (a missing row reads row 0, which exists whenever a tile does, and the value is
// discarded), so the loads of a stage are the same on every path and the wait before the MFMAs
// of a stage only covers that stage's loads, not the ones prefetched after it.
template <int KB, int NB, int MB, int KSPLIT>
__global__ __launch_bounds__(64 * KSPLIT) void conv_fwd_bf16_kernel(const uint16_t *__restrict__ X, int cin,
                                                                     const bf16x8_t *__restrict__ Wp,
                                                                     const float *__restrict__ bias, int cout,
                                                                     const int32_t *__restrict__ nbr,
                                                                     const npvs_counts *__restrict__ counts, int cap,
                                                                     int relu, int out_f32, void *__restrict__ Y) {
  constexpr int ROWS = 16 * MB;
  constexpr int KPER = 27 / KSPLIT;
  constexpr int NBLK = MB * NB;
  constexpr int S = KPER * KB;  // stages: (offset, 32-channel chunk)
  constexpr int PD = S < 4 ? S : 4;  // stages in flight
  static_assert(KPER * KSPLIT == 27, "KSPLIT must divide 27");
  __shared__ f32x4_t red[KSPLIT > 1 ? KSPLIT * NBLK * 64 : 1];
  const int32_t n = counts->n_sites;
  const int ntiles = (n + ROWS - 1) / ROWS;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index, uniform (scalar)
  const int kbeg = wv * KPER;
  // wide rows are gathered by pieces (512 -> 64, 1,802 sites: 28.2 us in the product's layout, 21.4 so);
  // one or two pieces a row are held, and the crossbar's latency shows
  constexpr bool PIECES = KB > 2;
  const int csub = PIECES ? piece_channel(lane) : 8 * (lane >> 4), grow = PIECES ? piece_row(lane) : lane & 15;
  for (int j = 0;; ++j) {
    const int tile = xcd_tile(blockIdx.x, gridDim.x, ntiles, j);
    if (tile < 0) break;
    const int row0 = tile * ROWS;
    const bf16x8_t *W = Wp + opaque_zero();
    int idx[KPER][MB];
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) idx[q][mb] = nbr_index(nbr, cap, kbeg + q, row0 + mb * 16 + grow, n);
    bool act[KPER];
#pragma unroll
    for (int q = 0; q < KPER; ++q) {
      bool a = false;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) a = a || idx[q][mb] >= 0;
      act[q] = __any(a);
    }
    f32x4_t acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8_t bx[PD][MB], aw[PD][NB];
#pragma unroll
    for (int st = -(PD - 1); st < S; ++st) {
      const int ld = st + PD - 1;  // stage whose loads are issued now
      if (ld < S) {  // compile-time after unrolling; loads are issued even for skipped offsets
        const int q = ld / KB, kb = ld % KB, slot = ld % PD;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) bx[slot][mb] = gather8(X, cin, idx[q][mb], kb * 32 + csub);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) aw[slot][nb] = W[(((int64_t)(kbeg + q) * NB + nb) * KB + kb) * 64 + lane];
      }
      if (st >= 0 && act[st / KB]) {
        const int slot = st % PD;
        bf16x8_t row[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          row[mb] = PIECES ? row_operand(__builtin_bit_cast(uint4, bx[slot][mb]), lane) : bx[slot][mb];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[slot][nb], row[mb], acc[mb][nb], 0, 0, 0);
      }
    }
    if constexpr (KSPLIT == 1) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          conv_bf16_epilogue<NB>(acc[mb][nb], row0 + mb * 16 + (lane & 15), n, nb * 16 + 4 * (lane >> 4), cout, bias,
                                 relu, out_f32, Y);
    } else {
      __syncthreads();  // the previous tile's readers are done with red
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) red[(wv * NBLK + mb * NB + nb) * 64 + lane] = acc[mb][nb];
      __syncthreads();
      for (int blk = wv; blk < NBLK; blk += KSPLIT) {
        f32x4_t sum = red[blk * 64 + lane];
        for (int w = 1; w < KSPLIT; ++w) sum += red[(w * NBLK + blk) * 64 + lane];
        const int mb = blk / NB, nb = blk % NB;
        conv_bf16_epilogue<NB>(sum, row0 + mb * 16 + (lane & 15), n, nb * 16 + 4 * (lane >> 4), cout, bias, relu,
                               out_f32, Y);
      }
    }
  }
}

// Shared-weight variant: the RG waves of a workgroup own different rows (16 MB each) and all 27
// offsets; each offset's packed weights are staged once per workgroup into a double-buffered LDS
// slot (loaded into registers one offset ahead, stored after the current offset's MFMAs), so the
// L2 reads of weights drop by a factor of RG.  The neighbour rows are gathered straight from
// global memory one offset ahead as in the split kernel.
// ------------------------------------------------------------------------------------------
// BF16 path for any channel counts (cin % 8 == 0, cout % 8 == 0), used for the shapes the tuned
// kernels above do not cover, e.g. the wide first and last layers of interleave factors 8 and 16
// (Cin or Cout = d^3 = 512 or 4096).  Workgroup = 9 waves over the same MB x 16 rows, wave w owning
// offsets 3w .. 3w + 2; blockIdx.z selects 64 output channels (4 MFMA output blocks).  The
// (offset, 32-channel chunk) stages are walked with a runtime chunk count and 4 stages in flight;
// loads past the last stage re-read it and are masked to zero, and offsets with no neighbour
// gather zeros, so every MFMA is unconditional (no branch around an accumulator).  The 9 partial
// sums are added in LDS in wave order, as in the split kernel.
// ------------------------------------------------------------------------------------------
// NBW: blocks of 16 outputs, 4, or 2 where no more are left of the workgroup's 64 (512 -> 32, 1,802 sites:
// 34.2 us with four, half of them repeats, 23.8 with two; 4,915 sites 46.9 and 34.0).
template <int MB, int NBW>
__device__ __forceinline__ void conv_bf16_wide_body(const uint16_t *__restrict__ X, int cin,
                                                    const bf16x8_t *__restrict__ Wp, const float *__restrict__ bias,
                                                    int cout, const int32_t *__restrict__ nbr, int n, int cap, int relu,
                                                    int out_f32, void *__restrict__ Y, float *__restrict__ part,
                                                    f32x4_t *__restrict__ red) {
  constexpr int KSPLIT = 9, KPER = 3, ROWS = 16 * MB, NBLK = MB * NBW, PD = MB > 2 ? 2 : 4;
  // by pieces, but for 16-row tiles: few workgroups then, and the crossbar is one more wait a stage (256 -> 64,
  // 1,024 sites: 19.4 us by pieces, 19.0 so)
  constexpr bool PIECES = MB > 1;
  const int ntiles = (n + ROWS - 1) / ROWS;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index, uniform (scalar)
  const int kbeg = wv * KPER, csub = PIECES ? piece_channel(lane) : 8 * (lane >> 4);
  const int grow = PIECES ? piece_row(lane) : lane & 15;
  const int KB = (cin + 31) / 32, NBT = (cout + 15) / 16, nb0 = 4 * blockIdx.z;
  // input-channel split (gridDim.x > 1 only with `part`): this workgroup's 32-channel chunks, at least one
  const int KBZ = (KB + gridDim.x - 1) / gridDim.x, kb_lo = blockIdx.x * KBZ;
  const int nkb = KB - kb_lo < KBZ ? KB - kb_lo : KBZ;
  const int S = KPER * nkb;  // stages of this wave
  for (int j = 0;; ++j) {
    int tile = blockIdx.y + j * gridDim.y;
    if (gridDim.x == 1) tile = xcd_tile(blockIdx.y, gridDim.y, ntiles, j);
    if (tile < 0 || tile >= ntiles) break;
    const int row0 = tile * ROWS;
    const bf16x8_t *W = Wp + opaque_zero();
    int idx[KPER][MB];
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) idx[q][mb] = nbr_index(nbr, cap, kbeg + q, row0 + mb * 16 + grow, n);
    f32x4_t acc[MB][NBW];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) acc[mb][nb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // the rows are held as loaded, with a mask that is applied where they are used: a mask at the load waits
    // for it, one round trip a stage
    uint4 bx[PD][MB];
    uint32_t bm[PD][MB];
    bf16x8_t aw[PD][NBW];
    // operands of stage st (clamped to the last one; zero rows past the end)
    auto load = [&](int st, int slot) {
      const bool live = st < S;
      st = live ? st : S - 1;
      const int q = st / nkb, kb = kb_lo + st - q * nkb;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int i = q == 0 ? idx[0][mb] : q == 1 ? idx[1][mb] : idx[2][mb];
        const int c = kb * 32 + csub;
        const bool ok = live && i >= 0 && c < cin;
        bx[slot][mb] = *reinterpret_cast<const uint4 *>(X + (ok ? (int64_t)i * cin + c : 0));
        bm[slot][mb] = ok ? ~0u : 0u;
      }
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) {
        const int g = nb0 + nb < NBT ? nb0 + nb : NBT - 1;  // blocks past cout: any valid fragment
        aw[slot][nb] = W[(((int64_t)(kbeg + q) * NBT + g) * KB + kb) * 64 + lane];
      }
    };
#pragma unroll
    for (int p = 0; p < PD; ++p) load(p, p);
    for (int g = 0; g < S; g += PD) {
#pragma unroll
      for (int p = 0; p < PD; ++p) {
        bf16x8_t row[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const uint4 v = bx[p][mb];
          const uint32_t m = bm[p][mb];
          const uint4 masked = make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
          row[mb] = PIECES ? row_operand(masked, lane) : __builtin_bit_cast(bf16x8_t, masked);
        }
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[p][nb], row[mb], acc[mb][nb], 0, 0, 0);
        load(g + p + PD, p);
      }
    }
    __syncthreads();  // the previous tile's readers are done with red
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) red[(wv * NBLK + mb * NBW + nb) * 64 + lane] = acc[mb][nb];
    __syncthreads();
    for (int blk = wv; blk < NBLK; blk += KSPLIT) {
      f32x4_t sum = red[blk * 64 + lane];
      for (int w = 1; w < KSPLIT; ++w) sum += red[(w * NBLK + blk) * 64 + lane];
      const int mb = blk / NBW, nb = blk % NBW;
      const int r = row0 + mb * 16 + (lane & 15), o = (nb0 + nb) * 16 + 4 * (lane >> 4);
      if (part) {  // raw partial sum of this channel range; the finishing kernel adds the ranges
        if (r < n && o < cout) *reinterpret_cast<f32x4_t *>(part + ((int64_t)blockIdx.x * cap + r) * cout + o) = sum;
      } else {
        conv_bf16_epilogue<4>(sum, r, n, o, cout, bias, relu, out_f32, Y);
      }
    }
  }
}

// MB = 1, 2 or 4 blocks of 16 rows per workgroup (equal sums either way); 0: by the number of sites.
// A workgroup reads all its weights once per tile, so more rows a tile read them less often, but fewer
// tiles leave CUs idle.  A round of 256 workgroups measured 23, 31 and 44 us for MB = 1, 2 and 4 (4096 ->
// 64 in 16 ranges, with the finishing launch), hence the least of 2, 3 and 4 times the rounds.  The range is
// blockIdx.x, so that ranges go to XCDs in turn and an XCD's L2 holds the weights of its own two of 16 (14 MB
// in all; 40 sites 47.2 us with a range's tiles over all XCDs, 21.6 so).  One block a tile before and this,
// 4096 -> 64, us: 397 sites 50.8 -> 31.3, 1,024 88.8 -> 43.8, 2,048 162.5 -> 82.5; 1024 -> 128, 1,802 sites
// 85.2 -> 42.3.
template <int MB>
__global__ __launch_bounds__(576) void conv_fwd_bf16_wide_kernel(const uint16_t *__restrict__ X, int cin,
                                                                  const bf16x8_t *__restrict__ Wp,
                                                                  const float *__restrict__ bias, int cout,
                                                                  const int32_t *__restrict__ nbr,
                                                                  const npvs_counts *__restrict__ counts, int cap,
                                                                  int relu, int out_f32, void *__restrict__ Y,
                                                                  float *__restrict__ part) {
  __shared__ f32x4_t red[9 * (MB ? MB : 4) * 4 * 64];
  const int32_t n = counts->n_sites;
  const bool half = cout - 64 * (int)blockIdx.z <= 32;
  auto body = [&](auto mb, auto nbw) {
    conv_bf16_wide_body<mb.value, nbw.value>(X, cin, Wp, bias, cout, nbr, n, cap, relu, out_f32, Y, part, red);
  };
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, 2> two{};
  constexpr std::integral_constant<int, 4> four{};
  if constexpr (MB > 0) {
    body(std::integral_constant<int, MB>{}, four);
  } else {
    const int split = gridDim.x * gridDim.z, t = (n + 15) / 16;
    const int c1 = 2 * ((t * split + 255) / 256), c2 = 3 * (((t + 1) / 2 * split + 255) / 256),
              c4 = 4 * (((t + 3) / 4 * split + 255) / 256);
    if (c1 <= c2 && c1 <= c4) {
      if (half) body(one, two);
      else body(one, four);
    } else if (c2 <= c4) {
      if (half) body(two, two);
      else body(two, four);
    } else {
      if (half) body(four, two);
      else body(four, four);
    }
  }
}

// Sum of the channel-range partials in range order, then bias, ReLU and rounding: one thread per
// 4 outputs of an active row.
__global__ __launch_bounds__(256) void conv_splitk_finish_kernel(const float *__restrict__ part, int KZ, int cap,
                                                                  const float *__restrict__ bias, int cout,
                                                                  const npvs_counts *__restrict__ counts, int relu,
                                                                  int out_f32, void *__restrict__ Y) {
  const int64_t q = cout / 4, total = (int64_t)counts->n_sites * q;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(e / q), o = (int)(e % q) * 4;
    f32x4_t sum = *reinterpret_cast<const f32x4_t *>(part + (int64_t)r * cout + o);
#pragma unroll 4
    for (int z = 1; z < KZ; ++z) sum += *reinterpret_cast<const f32x4_t *>(part + ((int64_t)z * cap + r) * cout + o);
    conv_bf16_epilogue<4>(sum, r, r + 1, o, cout, bias, relu, out_f32, Y);
  }
}

// ------------------------------------------------------------------------------------------
// BF16 path, weight-stationary, for inputs of at most 96 channels and any number of outputs.
// Workgroup = 9 waves over the same MB x 16 rows, wave w owning offsets 3w .. 3w + 2;
// blockIdx.y selects 16 NBW output channels (NBW MFMA output blocks).  A wave loads the weight
// fragments of its 3 offsets x KB chunks x NBW output blocks once and keeps them in registers
// while the workgroup walks its row tiles; the neighbour indices of the tile after next are
// loaded during the current tile.  The 9 partial sums are added in LDS in wave order.
// ------------------------------------------------------------------------------------------
// NBW: output blocks of 16 channels per workgroup (2, 4, or 1 for 4 or 5 input chunks).  With
// two blocks the rows of the next tile are gathered into a second buffer while the current
// tile's products run; with one or four (whose weights leave no registers for a second buffer)
// they are gathered into the same buffer as soon as the products have issued, ahead of the
// reduction and the epilogue.
// With FUSE (the data gradient of a layer, feeding the backward of the layer below): the result
// is masked by M > 0 (the ReLU' of the layer below, whose output M is; no mask when M is null),
// rounded to bf16 into Y, and each epilogue wave keeps per-lane running sums of its masked values
// over the tiles its workgroup walks; at the end a fixed butterfly adds the 16 rows of each
// column and workgroup b writes row b of the bias partial table dbp[kBwdDbBlocks][cout] (rows
// past the grid are written as zeros), so the layer below's bias gradient is a fixed-order sum
// over that table.  Needs one column group (cout <= 16 NBW) and MB = 1.
template <int KB, int MB, int NBW, bool FUSE>
__device__ __forceinline__ void wsta_body(const uint16_t *__restrict__ X, int cin, const bf16x8_t *__restrict__ Wp,
                                          const float *__restrict__ bias, int cout, const int32_t *__restrict__ nbr,
                                          const npvs_counts *__restrict__ counts, int cap, int relu, int out_f32,
                                          void *__restrict__ Y, const uint16_t *__restrict__ M,
                                          float *__restrict__ dbp) {
  constexpr int KSPLIT = 9, KPER = 3, ROWS = 16 * MB, NBLK = MB * NBW;
  constexpr bool PF = NBW == 2;  // rows of the next tile prefetched (the registers of 4 blocks' weights leave no room)
  static_assert(!FUSE || MB == 1, "the fused data gradient keeps one column block per epilogue wave");
  __shared__ f32x4_t red[KSPLIT * NBLK * 64];
  const int32_t n = counts->n_sites;
  const int ntiles = (n + ROWS - 1) / ROWS;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index, uniform (scalar)
  const int kbeg = wv * KPER, csub = 8 * (lane >> 4);
  const int NBT = (cout + 15) / 16, nb0 = NBW * blockIdx.y;
  bf16x8_t aw[KPER][KB][NBW];
#pragma unroll
  for (int q = 0; q < KPER; ++q)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) {
        const int g = nb0 + nb < NBT ? nb0 + nb : NBT - 1;  // blocks past cout: any valid fragment
        aw[q][kb][nb] = Wp[(((int64_t)(kbeg + q) * NBT + g) * KB + kb) * 64 + lane];
      }
  float da[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // FUSE: this lane's running column sums
  auto write_db_parts = [&]() {
    if (wv >= NBLK) return;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1)
#pragma unroll
      for (int i = 0; i < 4; ++i) da[i] += __shfl_xor(da[i], off, 64);
    const int o = (nb0 + wv) * 16 + 4 * (lane >> 4);
    if ((lane & 15) == 0 && o < cout)
      for (int row = blockIdx.x; row < kBwdDbBlocks; row += gridDim.x)
        *reinterpret_cast<f32x4_t *>(dbp + (int64_t)row * cout + o) =
            row == (int)blockIdx.x ? f32x4_t{da[0], da[1], da[2], da[3]} : f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  };
  int tile = xcd_tile(blockIdx.x, gridDim.x, ntiles, 0);
  if (tile < 0) {  // whole workgroup: tile depends on blockIdx only
    if constexpr (FUSE) write_db_parts();
    return;
  }
  // Loads retire in order, so a value used right after its load makes every load issued before
  // it wait too.  The neighbour indices are therefore loaded raw (rows past the last site read
  // the last site's entry) and judged only when their rows are gathered, and a gathered row is
  // loaded raw (a missing neighbour loads row 0) with its mask kept beside it, applied only where
  // the products read the row; the bias of the epilogue is loaded once, before the tiles.
  // (A missing tile re-reads the indices of the last valid one.)
  auto indices = [&](int t, int (&ix)[KPER][MB]) {
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int r = t * ROWS + mb * 16 + (lane & 15);
        ix[q][mb] = nbr[(int64_t)(kbeg + q) * cap + (r < n ? r : n - 1)];
      }
  };
  // rows of tile t, whose raw indices ix holds; bit q MB + mb of m marks a row that exists
  auto rows = [&](const int (&ix)[KPER][MB], int t, uint4 (&b)[KPER][KB][MB], uint32_t &m) {
    m = 0u;
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const bool ok = t * ROWS + mb * 16 + (lane & 15) < n && ix[q][mb] >= 0;
        m |= (ok ? 1u : 0u) << (q * MB + mb);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const int c = kb * 32 + csub;
          b[q][kb][mb] = *reinterpret_cast<const uint4 *>(X + (ok && c < cin ? (int64_t)ix[q][mb] * cin + c : 0));
        }
      }
  };
  auto masked = [&](const uint4 &v, uint32_t m, int bit, int kb) {
    const uint32_t mm = ((m >> bit) & 1u) && kb * 32 + csub < cin ? ~0u : 0u;
    return make_uint4(v.x & mm, v.y & mm, v.z & mm, v.w & mm);
  };
  // with a second buffer, rows are masked when they become the current tile's (a whole tile after
  // their loads were issued), so the current buffer needs no mask word
  auto mask_all = [&](const uint4 (&src)[KPER][KB][MB], uint32_t m, uint4 (&dst)[KPER][KB][MB]) {
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) dst[q][kb][mb] = masked(src[q][kb][mb], m, q * MB + mb, kb);
  };
  // the epilogue block of this wave (at most one: NBLK <= KSPLIT) and its bias, loaded once
  // (except with two 16-row blocks and a second row buffer, whose registers leave no room: there
  // the epilogue loads it, after this tile's loads and before the next tile's are needed)
  constexpr bool BIAS_ONCE = !(PF && MB == 2);
  float bv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (BIAS_ONCE && !FUSE) {
    const int o = (nb0 + wv % NBW) * 16 + 4 * (lane >> 4);
    if (bias && wv < NBLK && o < cout)
#pragma unroll
      for (int i = 0; i < 4; ++i) bv[i] = bias[o + i];
  }
  int ix[KPER][MB];
  uint4 bx[KPER][KB][MB];
  uint32_t bm;
  indices(tile, ix);
  rows(ix, tile, bx, bm);
  if constexpr (PF) mask_all(bx, bm, bx);
  int t1 = xcd_tile(blockIdx.x, gridDim.x, ntiles, 1);
  indices(t1 >= 0 ? t1 : tile, ix);
  for (int j = 0; tile >= 0; ++j) {
    const int t2 = xcd_tile(blockIdx.x, gridDim.x, ntiles, j + 2);
    // FUSE: the epilogue waves fetch this tile's mask before the next tile's rows are issued, so
    // waiting for it does not wait for them
    uint2 mk = {0u, 0u};
    if constexpr (FUSE) {
      const int r = tile * ROWS + (lane & 15), o = (nb0 + wv) * 16 + 4 * (lane >> 4);
      if (M && wv < NBLK && r < n && o < cout) mk = *reinterpret_cast<const uint2 *>(M + (int64_t)r * cout + o);
    }
    uint4 bn[KPER][KB][MB];
    uint32_t bnm;
    if constexpr (PF) {
      rows(ix, t1 >= 0 ? t1 : tile, bn, bnm);              // tile j + 1 (or a repeat)
      indices(t2 >= 0 ? t2 : (t1 >= 0 ? t1 : tile), ix);  // tile j + 2 (or a repeat)
    }
    f32x4_t acc[MB][NBW];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) acc[mb][nb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const uint4 row = PF ? bx[q][kb][mb] : masked(bx[q][kb][mb], bm, q * MB + mb, kb);
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[q][kb][nb], __builtin_bit_cast(bf16x8_t, row),
                                                                  acc[mb][nb], 0, 0, 0);
          }
    if constexpr (!PF) {
      // without a second row buffer, the next tile's rows go into this tile's registers as soon
      // as the products have taken them, their latency hidden by the reduction and the epilogue
      rows(ix, t1 >= 0 ? t1 : tile, bx, bm);               // tile j + 1 (or a repeat)
      indices(t2 >= 0 ? t2 : (t1 >= 0 ? t1 : tile), ix);  // tile j + 2 (or a repeat)
    }
    __syncthreads();  // the previous tile's readers are done with red
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) red[(wv * NBLK + mb * NBW + nb) * 64 + lane] = acc[mb][nb];
    __syncthreads();
    const int row0 = tile * ROWS;
    for (int blk = wv; blk < NBLK; blk += KSPLIT) {
      f32x4_t sum = red[blk * 64 + lane];
#pragma unroll 4  // with the next tile's rows in flight, a full unroll would spill
      for (int w = 1; w < KSPLIT; ++w) sum += red[(w * NBLK + blk) * 64 + lane];
      const int mb = blk / NBW, nb = blk % NBW;
      const int r = row0 + mb * 16 + (lane & 15), o = (nb0 + nb) * 16 + 4 * (lane >> 4);
      if constexpr (FUSE) {
        if (r < n && o < cout) {
          float g[4] = {sum[0], sum[1], sum[2], sum[3]};
          if (M) {
            const uint16_t mv[4] = {(uint16_t)mk.x, (uint16_t)(mk.x >> 16), (uint16_t)mk.y, (uint16_t)(mk.y >> 16)};
#pragma unroll
            for (int i = 0; i < 4; ++i) g[i] = bf16_to_f32(mv[i]) > 0.0f ? g[i] : 0.0f;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) da[i] += g[i];
          uint2 h;
          h.x = f32x2_to_bf16(g[0], g[1]);
          h.y = f32x2_to_bf16(g[2], g[3]);
          *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(Y) + (int64_t)r * cout + o) = h;
        }
      } else if constexpr (BIAS_ONCE) {
        conv_bf16_epilogue_bias(sum, r, n, o, cout, bv, relu, out_f32, Y);
      } else {
        conv_bf16_epilogue<4>(sum, r, n, o, cout, bias, relu, out_f32, Y);
      }
    }
    if constexpr (PF) {
      mask_all(bn, bnm, bx);
    }
    tile = t1;
    t1 = t2;
  }
  if constexpr (FUSE) write_db_parts();
}

// At most six waves a SIMD: with one input chunk two of the nine-wave workgroups then fit a compute unit, as
// the launch counts on, and not three, which leaves others one (32 -> 4096, 9,700 sites: 225 us with three, 200 with two).
template <int KB, int MB, int NBW = 2>
__global__ __launch_bounds__(576) __attribute__((amdgpu_waves_per_eu(3, 6))) void conv_fwd_bf16_wsta_kernel(const uint16_t *__restrict__ X, int cin,
                                                                  const bf16x8_t *__restrict__ Wp,
                                                                  const float *__restrict__ bias, int cout,
                                                                  const int32_t *__restrict__ nbr,
                                                                  const npvs_counts *__restrict__ counts, int cap,
                                                                  int relu, int out_f32, void *__restrict__ Y) {
  wsta_body<KB, MB, NBW, false>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, nullptr, nullptr);
}

// The weight-stationary layer (at most 64 outputs, 16-row tiles) with its cross-wave reduction
// taken off the product waves.  Nine product waves hold the weights of three offsets each and,
// per tile, write their partial products to one of two LDS tables; three reducer waves sum a
// table (partials 0 .. 8 in order, as the single-role kernel does) and apply the epilogue while
// the product waves go on to the next tile.  One barrier per tile: a table is rewritten two
// tiles later, after a barrier that every reducer reaches only once it has read the table.  The
// twelve waves fill three per SIMD at up to 168 registers, as many as the nine-wave kernel's
// register budget allows on the busiest SIMD.
// The gathered rows reach a product wave through LDS.  The MFMA operand wants lane l on row l % 16,
// and a load whose adjacent lanes lie on different rows takes one cycle per lane (67 cycles a KB),
// so each load instead covers whole rows with adjacent lanes (26 cycles a KB) and goes straight to
// a wave-private stage in LDS, one slot per offset; the operands are 16-byte LDS reads.  Everything
// runs one step ahead: while the products of tile j take offset q's operands, the slot of offset q
// (tile j + 1) is read into the same registers and then loaded again (tile j + 2), so the matrix
// cores, the LDS and the loads are busy at the same time.  The waits are counted by hand (a load to
// LDS has no register for the compiler to track); the product loop has no other load, because the
// reducers fetch the neighbour indices, six tiles ahead, into a ring in LDS.  A missing neighbour
// lies past the end of the row buffer and loads as zero, so no operand is masked.
// Measured, 64 -> 64, against rows loaded straight into registers: 9 699 rows 7.9 us (8.8), 20 971
// rows 11.3 (12.9), 140 078 rows 47.1 (51.8); 8 -> 64 on 49 283 rows 13.6 (15.5), 16 -> 16 on 819 rows
// 3.3 (3.7); vector instructions of the large layer 4.8 M against 11.2 M.  On the large
// layer the products of the SIMD with three product waves take 1 152 of a tile's 2 700 cycles, the
// loads 1 215 and the LDS about 1 400, and the barrier of each tile lets them overlap only in part.
template <int KB>
struct RowStage {
  static constexpr int LPR = 4 * KB;        // lanes (16-byte words) per row
  static constexpr int RPL = 64 / LPR;      // rows per load
  static constexpr int LOADS = 16 / RPL;    // loads per slot (16 rows of one offset)
  static constexpr int SLOT = 16 * LPR;     // 16-byte words per slot
  // word c of row r sits at place c ^ swz(r): the 8 lanes of one LDS pass, on consecutive rows at
  // one c, then fall on different banks
  static __device__ __forceinline__ int swz(int r) { return KB == 1 ? (r >> 1) & 3 : r & 7; }
};

// The rows X as a buffer of `bytes` bytes: a load past its end gives zero.
typedef int32_t rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_t row_buffer(const uint16_t *X, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(X);
  return rsrc_t{(int32_t)(uint32_t)a, (int32_t)((uint32_t)(a >> 32) & 0xffffu), (int32_t)bytes, 0x00020000};
}
// Start loads to LDS address dst (wave-uniform, bytes), lane i's 16 bytes (4 bytes) to dst + 16 i (4 i).
// No register is written: a load takes its LDS address from m0 and goes past the vector registers.
__device__ __forceinline__ void buffer_to_lds16(rsrc_t buf, uint32_t off, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(off), "s"(buf) : "memory");
}
__device__ __forceinline__ void global_to_lds4(const int32_t *src, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(dst), "v"(src) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {  // of a wave-uniform LDS pointer
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p);
}

// At most N of this wave's vector memory operations still in flight (in order: all older ones done).
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// This wave's LDS reads are in registers.
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// A workgroup barrier that orders LDS only: unlike __syncthreads it does not wait for loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// NBLK: output blocks of 16, 3 or 4.  With three, each reducer has one, and the
// fourth's products and partial sums, a repeat, are left out (24 -> 40, 115,343 sites: 24.2 us with four, 21.4).
template <int KB, int NBLK>
__global__ __launch_bounds__(768) void conv_fwd_bf16_wsred_kernel(const uint16_t *__restrict__ X, int cin,
                                                                  const bf16x8_t *__restrict__ Wp,
                                                                  const float *__restrict__ bias, int cout,
                                                                  const int32_t *__restrict__ nbr,
                                                                  const npvs_counts *__restrict__ counts, int cap,
                                                                  int relu, int out_f32, void *__restrict__ Y) {
  constexpr int KSPLIT = 9, KPER = 3, ROWS = 16, NRED = 3;
  constexpr int RING = 8, IDX = 512;  // ring slots; the 27 x 16 indices of a step, three loads of 64 a reducer
  typedef RowStage<KB> S;
  __shared__ f32x4_t red[2][KSPLIT * NBLK * 64];
  __shared__ uint4 stages[KSPLIT][KPER][S::SLOT];
  __shared__ int ring[RING][IDX];  // the neighbour indices [27][16] of step T's tile in slot T % RING
  const int32_t n = counts->n_sites;
  const int ntiles = (n + ROWS - 1) / ROWS;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index, uniform (scalar)
  const bool prod = wv < KSPLIT;                                     // a product wave (else a reducer)
  const int NBT = (cout + 15) / 16;
  const int tile0 = xcd_tile(blockIdx.x, gridDim.x, ntiles, 0);
  if (tile0 < 0) return;  // whole workgroup: tile depends on blockIdx only
  auto tile_at = [&](int j) { return xcd_tile(blockIdx.x, gridDim.x, ntiles, j); };
  // The two roles walk the same tiles in their own loops, one barrier per tile each (the role is
  // uniform over a wave, so every wave of the workgroup meets every barrier).
  if (prod) {
    // The first tile's rows are loaded straight into the operand registers, through this wave's own
    // index loads (a workgroup with one tile then needs nothing else); the second and third tiles'
    // indices are loaded here too, lane 16 q + r holding offset q, row r.
    const int kbeg = wv * KPER;
    auto own_index = [&](int k, int t) {  // rows past the last site take its neighbours: not stored
      const int r = t * ROWS + (lane & 15);
      return nbr[(int64_t)(kbeg + k) * cap + (r < n ? r : n - 1)];
    };
    int i0[KPER], i12[2] = {0, 0};
#pragma unroll
    for (int q = 0; q < KPER; ++q) i0[q] = own_index(q, tile0);
#pragma unroll
    for (int j = 1; j < 3; ++j)
      if (tile_at(j) >= 0) i12[j - 1] = own_index(lane < 48 ? lane >> 4 : 2, tile_at(j));
    bf16x8_t aw[KPER][KB][NBLK];
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int nb = 0; nb < NBLK; ++nb) {
          const int g = nb < NBT ? nb : NBT - 1;  // blocks past cout: any valid fragment
          aw[q][kb][nb] = Wp[(((int64_t)(kbeg + q) * NBT + g) * KB + kb) * 64 + lane];
        }
    // this lane's part of a slot's loads: rows t RPL + lane / LPR, always the same channels.  A
    // missing row (index -1, 2^24 - 1 as the 24 bits multiplied) and channels past cin lie past
    // the end of the buffer and load as zero.
    const rsrc_t rows = row_buffer(X, (uint32_t)n * (uint32_t)(2 * cin));  // at most 2^31 bytes: n < 2^24
    const int lr = lane / S::LPR, lc = 8 * ((lane % S::LPR) ^ S::swz(lr));
    const uint32_t coff = lc < cin ? 2 * lc : 0x80000000u;
    const uint32_t st0 = lds_address(stages[wv][0]);
    int src[KPER][S::LOADS];  // the rows of the step to load next
    auto indices = [&](int T) {
      const int *rs = ring[T % RING] + kbeg * ROWS + lr;
#pragma unroll
      for (int q = 0; q < KPER; ++q)
#pragma unroll
        for (int t = 0; t < S::LOADS; ++t) src[q][t] = rs[q * ROWS + t * S::RPL];
    };
    auto spread = [&](int ix) {  // the same from an index register of the prologue
#pragma unroll
      for (int q = 0; q < KPER; ++q)
#pragma unroll
        for (int t = 0; t < S::LOADS; ++t)
          src[q][t] = __builtin_amdgcn_ds_bpermute(4 * (q * ROWS + t * S::RPL + lr), ix);
    };
    auto load_slot = [&](int q) {
#pragma unroll
      for (int t = 0; t < S::LOADS; ++t)
        buffer_to_lds16(rows, __umul24((uint32_t)src[q][t], 2 * cin) + coff, st0 + 16 * (q * S::SLOT + t * 64));
    };
    bf16x8_t bx[KPER][KB];
    auto read_slot = [&](int q) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const int r = lane & 15, c = 4 * kb + (lane >> 4);
        bx[q][kb] = __builtin_bit_cast(bf16x8_t, stages[wv][q][r * S::LPR + (c ^ S::swz(r))]);
      }
    };
#pragma unroll
    for (int q = 0; q < KPER; ++q)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const int c = kb * 32 + 8 * (lane >> 4);
        bx[q][kb] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(X), 0, n * 2 * cin, 0x00020000),
            __umul24((uint32_t)i0[q], 2 * cin) + (c < cin ? 2 * c : 0x80000000u), 0, 0));
      }
    if (tile_at(1) >= 0) {
      spread(i12[0]);
#pragma unroll
      for (int q = 0; q < KPER; ++q) load_slot(q);
      spread(i12[1]);
    }
    // the weights and the first rows have landed: as the builtin, so that the compiler knows and
    // puts no wait for them (which would count the stage's loads) into the loop
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    // step j, with src the rows of step j + 2; MORE: how many steps follow (0, 1, or 2 for more)
    auto step = [&](int j, auto follow) {
      constexpr int MORE = decltype(follow)::value;
      f32x4_t acc[NBLK];
#pragma unroll
      for (int nb = 0; nb < NBLK; ++nb) acc[nb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int q = 0; q < KPER; ++q) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int nb = 0; nb < NBLK; ++nb)
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[q][kb][nb], bx[q][kb], acc[nb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE > 0) {
          wait_lds();  // slot q - 1 (and the indices) have been read
          if (MORE > 1 && q > 0) load_slot(q - 1);
          wait_loads<(MORE > 1 ? 2 * S::LOADS : 0)>();  // slot q holds step j + 1 (two slots' loads were issued after it)
          read_slot(q);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      f32x4_t *tab = red[j & 1];
#pragma unroll
      for (int nb = 0; nb < NBLK; ++nb) tab[(wv * NBLK + nb) * 64 + lane] = acc[nb];
      wait_lds();
      if constexpr (MORE > 1) load_slot(KPER - 1);
      lds_barrier();  // table j % 2 is complete
      if constexpr (MORE > 1) indices(j + 3);
    };
    int j = 0;
    for (; tile_at(j + 2) >= 0; ++j) step(j, std::integral_constant<int, 2>{});
    if (tile_at(j + 1) >= 0) step(j++, std::integral_constant<int, 1>{});
    step(j, std::integral_constant<int, 0>{});
  } else {
    const int rw = wv - KSPLIT, blk1 = rw + NRED;  // blocks rw and, for wave 9, blk1
    // this reducer's part of a step's indices, straight into the ring: entries rw + 3 u of 64 each
    // (entries past the 27 offsets repeat the last; rows past the last site take its neighbours:
    // their results are not stored)
    auto fetch = [&](int t, int T) {  // of tile t, step T
      const int r = t * ROWS + (lane & 15), rc = r < n ? r : n - 1;
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int g = rw + NRED * u, k = 4 * g + (lane >> 4);
        if (g < 7) global_to_lds4(nbr + (int64_t)(k < 27 ? k : 26) * cap + rc, lds_address(&ring[T % RING][64 * g]));
      }
    };
#pragma unroll
    for (int T = 3; T < 6; ++T)
      if (tile_at(T) >= 0) fetch(tile_at(T), T);
    float bv[2][4] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
    if (bias)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int blk = rw + NRED * h, o = blk * 16 + 4 * (lane >> 4);
        if (blk < NBLK && o < cout)
#pragma unroll
          for (int i = 0; i < 4; ++i) bv[h][i] = bias[o + i];
      }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), known to the compiler (the bias is used in the loop)
    // step j; `fetching`: there is a step j + 6, whose tile is t6
    auto step = [&](int j, int tile, int t6, auto fetching) {
      const f32x4_t *tab = red[j & 1];
      // the ring holds step j + 3, which the products read after this barrier: the loads of steps
      // j + 4 and j + 5 (two or three each) were issued after it
      wait_loads<(decltype(fetching)::value ? 4 : 0)>();
      lds_barrier();  // table j % 2 is complete; this wave is done with table (j - 1) % 2
      f32x4_t p0[KSPLIT], p1[KSPLIT];
#pragma unroll
      for (int w = 0; w < KSPLIT; ++w) p0[w] = tab[(w * NBLK + rw) * 64 + lane];
      if (blk1 < NBLK)
#pragma unroll
        for (int w = 0; w < KSPLIT; ++w) p1[w] = tab[(w * NBLK + blk1) * 64 + lane];
      if constexpr (decltype(fetching)::value) fetch(t6, j + 6);  // into the slot last read in step j - 5
      __builtin_amdgcn_sched_barrier(0);  // all in flight before any is added
      const int r = tile * ROWS + (lane & 15);
      f32x4_t sum = p0[0];
#pragma unroll
      for (int w = 1; w < KSPLIT; ++w) sum += p0[w];
      conv_bf16_epilogue_bias(sum, r, n, rw * 16 + 4 * (lane >> 4), cout, bv[0], relu, out_f32, Y);
      if (blk1 < NBLK) {
        sum = p1[0];
#pragma unroll
        for (int w = 1; w < KSPLIT; ++w) sum += p1[w];
        conv_bf16_epilogue_bias(sum, r, n, blk1 * 16 + 4 * (lane >> 4), cout, bv[1], relu, out_f32, Y);
      }
    };
    int j = 0, t = tile0;
    for (int t6 = tile_at(6); t6 >= 0; t6 = tile_at(++j + 6), t = tile_at(j)) step(j, t, t6, std::true_type{});
    for (; t >= 0; t = tile_at(++j)) step(j, t, 0, std::false_type{});
  }
}

// The data gradient of a BF16 layer with the ReLU' of the layer below fused in: dZ_below =
// bf16(conv(dZ, W') masked by M > 0) and the bias partial table dbp (see wsta_body).
template <int KB>
__global__ __launch_bounds__(576) void dgrad_relu_bf16_wsta_kernel(const uint16_t *__restrict__ dZ, int cin,
                                                                    const bf16x8_t *__restrict__ Wt, int cout,
                                                                    const int32_t *__restrict__ nbr,
                                                                    const npvs_counts *__restrict__ counts, int cap,
                                                                    uint16_t *__restrict__ dZ_below,
                                                                    const uint16_t *__restrict__ M,
                                                                    float *__restrict__ dbp) {
  wsta_body<KB, 1, 4, true>(dZ, cin, Wt, nullptr, cout, nbr, counts, cap, 0, 0, dZ_below, M, dbp);
}

template <int KB, int NB, int MB, int RG>
__global__ __launch_bounds__(64 * RG) void conv_fwd_bf16_lds_kernel(const uint16_t *__restrict__ X, int cin,
                                                                     const bf16x8_t *__restrict__ Wp,
                                                                     const float *__restrict__ bias, int cout,
                                                                     const int32_t *__restrict__ nbr,
                                                                     const npvs_counts *__restrict__ counts, int cap,
                                                                     int relu, int out_f32, void *__restrict__ Y) {
  constexpr int ROWS = 16 * MB * RG;
  constexpr int FR = NB * KB;              // weight fragments of one offset (64 lanes x 16 bytes each)
  constexpr int WPT = (FR + RG - 1) / RG;  // fragments each thread stages per offset (some idle)
  constexpr int NS = 4;                    // LDS weight slots: offset o lives in slot o % NS
  // Offset o's weights are loaded into registers at step o - 4, stored to LDS at step o - 2 and
  // read at step o; its rows are gathered at step o - 3.  One barrier ends every step, which
  // orders each slot's store after the last read of the offset it held (step o - 4) and before
  // its first read.
  __shared__ bf16x8_t Ws[NS][FR * 64];
  const int32_t n = counts->n_sites;
  const int ntiles = (n + ROWS - 1) / ROWS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform (scalar)
  const int csub = 8 * (lane >> 4);
  for (int j = 0;; ++j) {
    const int tile = xcd_tile(blockIdx.x, gridDim.x, ntiles, j);
    if (tile < 0) break;
    const int row0 = tile * ROWS + wv * 16 * MB;
    const bf16x8_t *W = Wp + opaque_zero();
    int idx[27][MB];
#pragma unroll
    for (int q = 0; q < 27; ++q)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) idx[q][mb] = nbr_index(nbr, cap, q, row0 + mb * 16 + (lane & 15), n);
    f32x4_t acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8_t wreg[2][WPT], bx[4][MB][KB];
    auto wload = [&](int o, bf16x8_t (&w)[WPT]) {
#pragma unroll
      for (int i = 0; i < WPT; ++i)
        if (FR % RG == 0 || tid + i * 64 * RG < FR * 64) w[i] = W[(int64_t)o * FR * 64 + tid + i * 64 * RG];
    };
    auto wstore = [&](int slot, const bf16x8_t (&w)[WPT]) {
#pragma unroll
      for (int i = 0; i < WPT; ++i)
        if (FR % RG == 0 || tid + i * 64 * RG < FR * 64) Ws[slot][tid + i * 64 * RG] = w[i];
    };
    auto gather = [&](int o, bf16x8_t (&b)[MB][KB]) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) b[mb][kb] = gather8(X, cin, idx[o][mb], kb * 32 + csub);
    };
    // prologue: offsets 0 and 1 in LDS, 2 and 3 in registers, rows of offsets 0-2
    {
      bf16x8_t w0[WPT], w1[WPT];
      wload(0, w0);
      wload(1, w1);
      wload(2, wreg[0]);
      wload(3, wreg[1]);
      gather(0, bx[0]);
      gather(1, bx[1]);
      gather(2, bx[2]);
      wstore(0, w0);
      wstore(1, w1);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 27; ++k) {
      if (k + 2 < 27) wstore((k + 2) % NS, wreg[k % 2]);  // offset k + 2 (loaded at step k - 2)
      if (k + 4 < 27) wload(k + 4, wreg[k % 2]);
      if (k + 3 < 27) gather(k + 3, bx[(k + 3) % 4]);
      // offsets without any neighbour in this wave gather zeros: no branch around the products
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const bf16x8_t aw = Ws[k % NS][(nb * KB + kb) * 64 + lane];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw, bx[k % 4][mb][kb], acc[mb][nb], 0, 0, 0);
        }
      __syncthreads();
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        conv_bf16_epilogue<NB>(acc[mb][nb], row0 + mb * 16 + (lane & 15), n, nb * 16 + 4 * (lane >> 4), cout, bias,
                               relu, out_f32, Y);
  }
}

template <int KB, int NB, int MB, int RG>
static void launch_bf16_lds(const void *X, int cin, const void *Wp, const float *bias, int cout, const int32_t *nbr,
                            const npvs_counts *counts, int cap, int relu, int out_f32, void *Y, hipStream_t s) {
  int G = stride_grid(cap, 16 * MB * RG, 4096);
  G = (G + 7) & ~7;
  conv_fwd_bf16_lds_kernel<KB, NB, MB, RG><<<G, 64 * RG, 0, s>>>(
      (const uint16_t *)X, cin, (const bf16x8_t *)Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y);
}

// Tile shapes.  Split kernel (MB, KSPLIT) = (rows per wave / 16, waves sharing the 27 offsets of a
// tile): variant 0 (1, 9), 1 (2, 1), 2 (1, 3), 3 (2, 3), 4 (1, 1), 5 (2, 9).  Shared-weight kernel
// (MB, RG) = (rows per wave / 16, waves per workgroup): 6 (1, 4), 7 (1, 2), 8 (2, 2), 9 (1, 8),
// 10 (2, 4), 11 (2, 8).  Larger row blocks read each staged weight fragment for more rows (less
// weight traffic per row) and suit large batches; small ones keep more waves busy on one frame.
// Weight-stationary kernel (inputs of at most 64 channels): 12 (16-row tiles), 13 (32-row tiles).
// Inputs wider than 64 channels use only the 9-way split (a long unrolled offset loop would not
// fit the registers, nor a double-buffered offset of weights the LDS).
// kDefaultConvVariant is used by npvs_sparse_conv_fwd; the autotuner can pick another per layer.

template <int KB, int NB, int MB, int KSPLIT>
static void launch_bf16(const void *X, int cin, const void *Wp, const float *bias, int cout, const int32_t *nbr,
                        const npvs_counts *counts, int cap, int relu, int out_f32, void *Y, hipStream_t s) {
  const int rows = 16 * MB;
  int G = stride_grid(cap, rows, 4096);
  G = (G + 7) & ~7;
  conv_fwd_bf16_kernel<KB, NB, MB, KSPLIT><<<G, 64 * KSPLIT, 0, s>>>(
      (const uint16_t *)X, cin, (const bf16x8_t *)Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y);
}

template <int KB, int MB, int NBW = 2>
static void launch_bf16_wsta(const void *X, int cin, const void *Wp, const float *bias, int cout, const int32_t *nbr,
                             const npvs_counts *counts, int cap, int relu, int out_f32, void *Y, hipStream_t s) {
  // as many workgroups as fit on the chip at once (9-wave workgroups: two per compute unit with
  // one input chunk, one with two or more chunks or 32-row tiles), spread over the output groups;
  // each walks several row tiles
  const int groups = (cout + 16 * NBW - 1) / (16 * NBW);
  int G = (KB == 1 && MB == 1 && NBW <= 2 ? 512 : 256) / groups;
  G = G < 8 ? 8 : G & ~7;  // a multiple of 8 (one per XCD), rounded down so that all fit at once
  const int most = stride_grid(cap, 16 * MB, 4096);
  if (G > most) G = (most + 7) & ~7;
  conv_fwd_bf16_wsta_kernel<KB, MB, NBW><<<dim3(G, groups), 576, 0, s>>>(
      (const uint16_t *)X, cin, (const bf16x8_t *)Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y);
}

npvs_status dgrad_relu_fused(const uint16_t *dZ, int cin, const void *Wt, int cout, const int32_t *nbr,
                             const npvs_counts *counts, int cap, const uint16_t *M, uint16_t *dZ_below, float *dbp,
                             hipStream_t s) {
  if (cin > 64 || cin % 8 || cout > 64 || cout % 4)
    return fail(NPVS_ERR_UNSUPPORTED, "data gradient with fused ReLU': unsupported channel counts");
  // the grid of the default forward shape (one column group); at most kBwdDbBlocks workgroups,
  // one bias partial row each
  int G = 256;
  const int most = stride_grid(cap, 16, 4096);
  if (G > most) G = (most + 7) & ~7;
  G = G > kBwdDbBlocks ? kBwdDbBlocks : G;
  const bf16x8_t *W = (const bf16x8_t *)Wt;
  if (cin <= 32)
    dgrad_relu_bf16_wsta_kernel<1><<<dim3(G, 1), 576, 0, s>>>(dZ, cin, W, cout, nbr, counts, cap, dZ_below, M, dbp);
  else
    dgrad_relu_bf16_wsta_kernel<2><<<dim3(G, 1), 576, 0, s>>>(dZ, cin, W, cout, nbr, counts, cap, dZ_below, M, dbp);
  return check_hip(hipGetLastError(), "data gradient with fused ReLU'");
}

template <int MB>
static void launch_bf16_wide(const void *X, int cin, const void *Wp, const float *bias, int cout, const int32_t *nbr,
                             const npvs_counts *counts, int cap, int relu, int out_f32, void *Y, hipStream_t s,
                             int KZ, float *part) {
  const int groups = (cout + 63) / 64, split = (part ? KZ : 1) * groups;
  // one workgroup per CU, which walks its tiles: the capacity's tiles would launch several rounds of
  // workgroups past the sites, each with the LDS of a CU (4096 -> 64, 397 sites of 2,048: 48.5 us, 31.3 so).
  // At least eight tiles are walked at once (one per XCD), so that more than 32 ranges times groups, such as
  // 4096 -> 512 or 168 -> 4096, do take several rounds.
  const int G = (stride_grid(cap, 16 * (MB ? MB : 1), 256 / split > 8 ? 256 / split : 8) + 7) & ~7;
  const dim3 grid(part ? KZ : 1, G, groups);
  conv_fwd_bf16_wide_kernel<MB><<<grid, 576, 0, s>>>((const uint16_t *)X, cin, (const bf16x8_t *)Wp, bias, cout, nbr,
                                                      counts, cap, relu, out_f32, Y, part);
  if (part)
    conv_splitk_finish_kernel<<<stride_grid((int64_t)cap * (cout / 4), 256, 4096), 256, 0, s>>>(
        part, KZ, cap, bias, cout, counts, relu, out_f32, Y);
}

template <int KB, int NB>
static void launch_bf16_variant(int v, const void *X, int cin, const void *Wp, const float *bias, int cout,
                                const int32_t *nbr, const npvs_counts *counts, int cap, int relu, int out_f32, void *Y,
                                hipStream_t s) {
  if constexpr (KB > 2) {
    if (v == 5)
      launch_bf16<KB, NB, 2, 9>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    else
      launch_bf16<KB, NB, 1, 9>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
  } else {
    switch (v) {
      case 0: launch_bf16<KB, NB, 1, 9>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 1: launch_bf16<KB, NB, 2, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 2: launch_bf16<KB, NB, 1, 3>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 3: launch_bf16<KB, NB, 2, 3>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 4: launch_bf16<KB, NB, 1, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 5: launch_bf16<KB, NB, 2, 9>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 6: launch_bf16_lds<KB, NB, 1, 4>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 7: launch_bf16_lds<KB, NB, 1, 2>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 8: launch_bf16_lds<KB, NB, 2, 2>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 9: launch_bf16_lds<KB, NB, 1, 8>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      case 10: launch_bf16_lds<KB, NB, 2, 4>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
      default: launch_bf16_lds<KB, NB, 2, 8>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); break;
    }
  }
}

}  // namespace npvs

using namespace npvs;

extern "C" size_t npvs_packed_weight_bytes(int32_t cin, int32_t cout, int32_t dtype) {
  if (cin < 1 || cout < 1) return 0;
  if (dtype == NPVS_F32) return sizeof(float) * 27 * (size_t)cin * cout;
  if (dtype == NPVS_BF16) {
    size_t a = 27 * (size_t)((cout + 15) / 16) * ((cin + 31) / 32) * 1024;
    size_t b = 27 * (size_t)((cin + 15) / 16) * ((cout + 31) / 32) * 1024;
    return a > b ? a : b;
  }
  return 0;
}

extern "C" npvs_status npvs_pack_weights(const float *W, int32_t cin, int32_t cout, int32_t dtype,
                                        int32_t flip_transpose, void *Wp, void *stream) {
  if (!W || !Wp) return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights: null pointer");
  if (cin < 1 || cout < 1) return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights: channels must be >= 1");
  hipStream_t s = as_stream(stream);
  if (dtype == NPVS_F32) {
    pack_f32_kernel<<<stride_grid(27LL * cin * cout, 256, 1024), 256, 0, s>>>(W, cin, cout, flip_transpose ? 1 : 0,
                                                                             (float *)Wp);
  } else if (dtype == NPVS_BF16) {
    const int64_t buf = (int64_t)npvs_packed_weight_bytes(cin, cout, dtype) / 2;
    pack_bf16_kernel<<<stride_grid(buf, 256, 1024), 256, 0, s>>>(W, cin, cout, flip_transpose ? 1 : 0, buf,
                                                                  (uint16_t *)Wp);
  } else {
    return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights: dtype must be NPVS_F32 or NPVS_BF16");
  }
  return check_hip(hipGetLastError(), "npvs_pack_weights");
}

extern "C" npvs_status npvs_pack_weights_batch(int32_t n, const npvs_pack_desc *descs, int32_t dtype, void *stream) {
  if (n < 0 || n > NPVS_MAX_PACK) return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights_batch: n out of range");
  if (n == 0) return NPVS_OK;
  if (!descs) return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights_batch: null descriptors");
  if (dtype != NPVS_F32 && dtype != NPVS_BF16)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights_batch: dtype must be NPVS_F32 or NPVS_BF16");
  PackBatch PB = {};
  size_t most = 0;
  for (int i = 0; i < n; ++i) {
    const npvs_pack_desc &D = descs[i];
    if (!D.W || !D.Wp) return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights_batch: null pointer");
    if (D.cin < 1 || D.cout < 1) return fail(NPVS_ERR_INVALID_ARG, "npvs_pack_weights_batch: channels must be >= 1");
    PB.d[i] = D;
    const size_t e = npvs_packed_weight_bytes(D.cin, D.cout, dtype) / (dtype == NPVS_F32 ? 4 : 2);
    PB.elems[i] = (int64_t)e;
    most = e > most ? e : most;
  }
  dim3 grid(stride_grid((int64_t)most, 256, 256), n);
  pack_batch_kernel<<<grid, 256, 0, as_stream(stream)>>>(PB, dtype);
  return check_hip(hipGetLastError(), "npvs_pack_weights_batch");
}

namespace npvs {
// Input-channel split of the general BF16 kernel: 1, or the number of ranges for 1024+ input channels
// (at most 16, of ceil(KB / wanted) chunks of 32 channels each but the last).  The ranges are counted from
// their length, so that none is empty: 16 wanted ranges of 129 chunks have 9 chunks each, which 15 ranges
// cover.  A workgroup of an empty range would divide by its chunk count of zero and, where the count is
// negative, address weights past the last offset's.
int splitk_factor(int32_t cin, int32_t cout, int32_t dtype) {
  const int KB = (cin + 31) / 32;
  if (dtype != NPVS_BF16 || KB < 32 || cin % 8 || cout % 8) return 1;
  const int wanted = KB / 8 > 16 ? 16 : KB / 8, len = (KB + wanted - 1) / wanted;
  return (KB + len - 1) / len;
}

size_t conv_fwd_ws_bytes(int32_t cin, int32_t cout, int32_t cap, int32_t dtype) {
  const int kz = splitk_factor(cin, cout, dtype);
  return kz > 1 ? sizeof(float) * (size_t)kz * cap * cout : 0;
}

// Dispatch by type, variant and (ceil(cin / 32), ceil(cout / 16)).
npvs_status conv_fwd_dispatch(const void *X, int32_t cin, const void *Wp, const float *bias, int32_t cout,
                              const int32_t *nbr, const npvs_counts *counts, int32_t cap, int32_t dtype, int32_t relu,
                              int32_t out_f32, void *Y, hipStream_t s, int variant, void *ws, size_t ws_bytes) {
  if (dtype == NPVS_F32) {
    // output blocks of 16 in groups of at most 4, as even as they divide
    const int blocks = (cout + 15) / 16, per = (blocks + 3) / 4, NI = (blocks + per - 1) / per;
    const float *Xf = static_cast<const float *>(X), *P = static_cast<const float *>(Wp);
    float *Yf = static_cast<float *>(Y);
    switch (NI) {
      case 1: launch_conv_f32<1>(Xf, cin, P, bias, cout, nbr, counts, cap, relu, Yf, s); break;
      case 2: launch_conv_f32<2>(Xf, cin, P, bias, cout, nbr, counts, cap, relu, Yf, s); break;
      case 3: launch_conv_f32<3>(Xf, cin, P, bias, cout, nbr, counts, cap, relu, Yf, s); break;
      default: launch_conv_f32<4>(Xf, cin, P, bias, cout, nbr, counts, cap, relu, Yf, s); break;
    }
    return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
  }
  if (cin % 8 || cout % 8)
    return fail(NPVS_ERR_UNSUPPORTED, "npvs_sparse_conv_fwd: BF16 needs cin % 8 == 0 and cout % 8 == 0");
  const int KB = (cin + 31) / 32, NB = (cout + 15) / 16;
  if (variant == 15) {  // variant 14 with dedicated reducer waves: at most 64 inputs and outputs
    // (row indices are 24 bits there).  At most 32 inputs and 32 outputs: the single-role shape of 32
    // outputs, two workgroups of which fit a CU, while the staged copies cost the same however few
    // channels a row has (8 -> 8, us, staged / single-role: 9,175 sites 5.3 / 4.7, 52,428 12.7 / 9.3,
    // 115,343 24.1 / 16.0; 32 -> 32 5.5 / 4.9, 13.3 / 10.0, 25.5 / 18.1).  With 33 to 48 outputs that
    // shape takes two groups of workgroups: 24 -> 40 4.8 / 6.4, 11.4 / 15.8, 21.4 / 29.6.
    if (KB == 1 && NB <= 2) {
      launch_bf16_wsta<1, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
      return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
    }
    // The copies to LDS take rows at 16-byte boundaries only; rows that lie between (a slice of a buffer
    // from an odd element on) take variant 14, whose loads to registers read from any address.
    if (KB <= 2 && NB <= 4 && cap < (1 << 24) && (reinterpret_cast<uintptr_t>(X) & 15) == 0) {
      int G = 256;
      const int most = stride_grid(cap, 16, 4096);
      if (G > most) G = (most + 7) & ~7;
      auto launch = [&](auto kernel) {
        kernel<<<dim3(G, 1), 768, 0, s>>>((const uint16_t *)X, cin, (const bf16x8_t *)Wp, bias, cout, nbr, counts, cap,
                                          relu, out_f32, Y);
      };
      if (KB == 2) launch(conv_fwd_bf16_wsred_kernel<2, 4>);
      else if (NB == 4) launch(conv_fwd_bf16_wsred_kernel<1, 4>);
      else launch(conv_fwd_bf16_wsred_kernel<1, 3>);
      return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
    }
    variant = 14;
  }
  if (variant == 14 && KB <= 2 && NB <= 4) {  // weight-stationary, all (at most 64) outputs per workgroup
    if (KB == 1) launch_bf16_wsta<1, 1, 4>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    else launch_bf16_wsta<2, 1, 4>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
  }
  if (variant == 14) variant = 12;  // more than 64 outputs: 32 per workgroup
  if ((variant == 12 || variant == 13) && KB <= 2) {  // weight-stationary tiles
    if (KB == 1) {
      if (variant == 12) launch_bf16_wsta<1, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
      else launch_bf16_wsta<1, 2>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    } else {
      if (variant == 12) launch_bf16_wsta<2, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
      else launch_bf16_wsta<2, 2>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    }
    return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
  }
#define NPVS_BF16_CASE(kb, nb)                                                                           \
  if (KB == kb && NB == nb) {                                                                            \
    launch_bf16_variant<kb, nb>(variant, X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s); \
    return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");                                         \
  }
  NPVS_BF16_CASE(1, 1)
  NPVS_BF16_CASE(1, 2)
  NPVS_BF16_CASE(1, 3)
  NPVS_BF16_CASE(1, 4)
  NPVS_BF16_CASE(2, 1)
  NPVS_BF16_CASE(2, 2)
  NPVS_BF16_CASE(2, 3)
  NPVS_BF16_CASE(2, 4)
  NPVS_BF16_CASE(16, 4)
#undef NPVS_BF16_CASE
  // any other shape: up to 64 input channels (e.g. the wide last layer of d = 8 or 16) the
  // weight-stationary kernel, else the general one (variants 5 and 13 pick 32-row tiles)
  if (KB <= 2) {
    const bool wide_rows = variant == 5 || variant == 13;
    if (KB == 1) {
      if (wide_rows) launch_bf16_wsta<1, 2>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
      else launch_bf16_wsta<1, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    } else {
      if (wide_rows) launch_bf16_wsta<2, 2>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
      else launch_bf16_wsta<2, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    }
    return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
  }
  // 65 to 160 input channels (the U-Net decoder: 160 -> 96, 96 -> 96, 96 -> 64): the
  // weight-stationary kernel, since the general kernel re-reads every offset's weights for each
  // 16-row tile; 3 input chunks with two output blocks per workgroup (168 VGPRs), 4 or 5 with one
  if (KB <= 5 && variant != 5) {
    if (KB == 3) launch_bf16_wsta<3, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    else if (KB == 4) launch_bf16_wsta<4, 1, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    else launch_bf16_wsta<5, 1, 1>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s);
    return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
  }
  // wide inputs: split the channel chunks over workgroups when the caller gave a workspace
  const int KZ = splitk_factor(cin, cout, dtype);
  float *part = (KZ > 1 && ws && ws_bytes >= conv_fwd_ws_bytes(cin, cout, cap, dtype)) ? (float *)ws : nullptr;
  if (variant == 5 || variant == 13)
    launch_bf16_wide<2>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s, KZ, part);
  else
    launch_bf16_wide<0>(X, cin, Wp, bias, cout, nbr, counts, cap, relu, out_f32, Y, s, KZ, part);
  return check_hip(hipGetLastError(), "npvs_sparse_conv_fwd");
}
}  // namespace npvs

extern "C" npvs_status npvs_conv_fwd_workspace_size(int32_t cin, int32_t cout, int32_t cap_sites, int32_t dtype,
                                                    size_t *bytes) {
  if (!bytes || cin < 1 || cout < 1 || cap_sites < 1)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_conv_fwd_workspace_size: bad arguments");
  *bytes = conv_fwd_ws_bytes(cin, cout, cap_sites, dtype);
  return NPVS_OK;
}

extern "C" npvs_status npvs_sparse_conv_fwd(const void *X, int32_t cin, const void *Wp, const float *bias,
                                           int32_t cout, const int32_t *nbr, const npvs_counts *counts,
                                           int32_t cap_sites, int32_t dtype, int32_t relu, int32_t out_f32,
                                           int32_t variant, void *Y, void *ws, size_t ws_bytes, void *stream) {
  if (!X || !Wp || !nbr || !counts || !Y) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_fwd: null pointer");
  if (cin < 1 || cout < 1 || cap_sites < 1) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_fwd: bad sizes");
  if (dtype != NPVS_F32 && dtype != NPVS_BF16)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_fwd: dtype must be NPVS_F32 or NPVS_BF16");
  if (X == Y) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_fwd: X and Y must not alias");
  if (variant == -1) variant = kDefaultConvVariant;
  if (variant < 0 || variant >= NPVS_CONV_VARIANTS)
    return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_fwd: variant out of range");
  const size_t need = conv_fwd_ws_bytes(cin, cout, cap_sites, dtype);
  if (ws && ws_bytes < need) return fail(NPVS_ERR_INVALID_ARG, "npvs_sparse_conv_fwd: workspace too small");
  return conv_fwd_dispatch(X, cin, Wp, bias, cout, nbr, counts, cap_sites, dtype, relu, out_f32, Y,
                           as_stream(stream), variant, ws, ws ? ws_bytes : 0);
}
