// Latent-space neighbourhoods B_k(x) of every code of a VQ codebook (paper
// Sec. 2.2: the k nearest neighbours of a token in latent space; reused by Sec. 4).
//
// The result is defined by the float64 inner product (products added in index
// order) with ties to the lower index, so it does not depend on how the matrix
// cores round.  The V x V similarities are never written out and the float64 keys
// are only formed where they decide something:
//   stats    norms, 1-norms, largest magnitude, halves of short rows, a padded copy where rows do not start on 16 bytes
//   limbs    (rows of more than 16 floats) fixed-point image of the codebook as three
//            8-bit limbs, in matrix-core fragment order
//   sample   per row: histogram of its similarities with a hashed, stratified sample of
//            about 4096 codes; the threshold is the sample's quantile at which, five
//            standard deviations of the sample's share allowed, k - 1 codes lie above (short rows: its
//            bin looked at again in 1024 parts where a few codes far longer than the rest crowd the others into it)
//   collect  the dense V x V contraction on the matrix cores, once (long rows: its half, it is symmetric): every code above the
//            row's threshold is appended to its list as one 32-bit word, similarity
//            (fixed point) over code index
//   rank     per row: the list is sorted by its approximate similarities (value buckets in
//            LDS); entries whose similarities differ by less than twice the bound on
//            their error are ordered by their exact float64 keys (long rows: by float64 sums in any order where these
//            are far enough apart), everything else already is
//   exact    rows that their list does not decide, over all codes (a launch of its own where that pays)
// Small codebooks of short rows (V <= kDirectCodes, D <= 16) take one kernel that does all of it.
//
// Why the list is enough: an outsider's similarity is at most threshold + e, e bounding the error of
// an approximate similarity.  If the (k-1)-th largest approximate similarity of the list exceeds
// the threshold by more than 2 e, the k - 1 largest all exceed every outsider.  Rows that fail this
// test, overflow their list or hold fewer than k - 1 entries (a sample that misleads, heavy ties)
// take an exact, slow radix select over all V codes instead.
//
// The approximate similarities and their bound e:
//   rows of up to 16 floats: x = h + l in halves of 11 bits, h h' + l h' + h l' on the f16 matrix
//   cores; what is left out is below 3 2^-22 |e_i| |e_j|.  The products are exact in float32; that each of
//   the additions, 32 N at most, is off by at most 2^-23 of |e_i| |e_j| is how the matrix cores are taken to add, not
//   something their documents promise.  (24 N products are not zero by construction.  The collecting sweep adds up 64 for either N, the
//   sample 32 N; the others are exact zeros, which round nothing.)  The halves are of 4096 x, or of 4 x in codebooks with entries from 16 on;
//   from 16376 on every row takes the exact path.
//   longer rows: x = q D + d with a 24-bit integer q = 2^16 a + 2^8 b + c (a, b, c signed 8-bit
//   limbs), |d| <= D / 2, D = largest magnitude / (127 2^16).  All limb products but c c are summed
//   exactly in int32 by the i8 matrix cores (eight MFMA 16x16x64 per 64 dimensions), so the only
//   errors are the quantisation, D/2 (|e_i|_1 + |e_j|_1), and a few units of the last place kept.
//   This is far tighter than what can be proved for fp32 accumulation of the same rows, at four times
//   its rate; at unit rows of 256 floats about one entry in twenty needs a float64 sum, hardly one its key.
#include <limits.h>
#include <math.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "lpp_internal.h"
#include "lpp_knn_list.h"

namespace {

// x, as something the compiler does not know: what is formed from it is formed here, and takes no registers before.
__device__ __forceinline__ int formed_anew(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kShortRow = 16;                 // rows of up to this many floats: pairs of halves
constexpr int kDirectCodes = 1024;            // codebooks of short rows up to this size: one kernel
constexpr int kLaterCodes = 4096;             // (see the rule at the end of this file)
constexpr int kLaterFloats = 1 << 20;
constexpr int kSampleCodes = 4096;            // codes a row's threshold is estimated from
constexpr int kSampleBins = 1024;             // bins of the estimate, [-|e_i| max|e_j|, +]
constexpr int kSampleThreads = 1024;
constexpr int kCollectWaves = 4;              // (long rows) waves per block
constexpr int kStatBlocks = 256, kStatThreads = 1024;
constexpr float kHalfScale = 4096.0f;         // short rows as halves: entries below 15.9
constexpr float kWideScale = 4.0f;            // ... of codebooks with larger ones: below 16376
constexpr float kLimbRange = 8323072.0f;      // 127 * 2^16: the largest |q|

// What the collecting kernel needs of a row: a code passes where d = similarity - thr is not negative, and
// leaves min(d a, qmax) (short rows: in float32, in the units of the scaled halves; long rows: int32, units
// of 2^24 unit^2).  E: entries whose left values differ by at most E may be in either order.
struct RowPlan {
  float a;
  union { float thr; int32_t thr_u; };
  int32_t E;
  int32_t flags;                              // kAll: every code passes; kAnyNan: some code holds a NaN; kNoList: exact path;
                                              // kFlat: its similarities are all the same; kWide: halves of kWideScale
};
constexpr int kAll = 1, kAnyNan = 2, kNoList = 4, kFlat = 8, kWide = 16;
// Rows of up to this many floats, more of a list's entries than an eighth of the threads being near ties: a thread forms an
// entry's key, a chain that short costs less than the sums and their comparison (every code four times, 4096 x 64,
// k = 300: 91 us and 162).  Few entries: the chain's loads in turn cost more (2000 x 64, k = 50: 37.4 us and 36.2).
constexpr int kChainFloats = 64;
constexpr int kMaxSplits = 16;                // (long rows) blocks that share a group's tiles
constexpr int kUnits = 256;                   // compute units of the card these kernels are for
constexpr size_t kMostLds = 150 * 1024;       // dynamic LDS of a block, static arrays beside it

struct KnnArgs {
  const float* E;
  int32_t V, D, k;
  int32_t PD;           // floats per row of Ep: D rounded up to 4
  int32_t Vp;           // V rounded up to 128
  int32_t cap;          // entries a row's list holds
  int32_t ib;           // index bits of a list word; 32 - ib value bits (at most 24)
  int32_t vmask_bits;   // value bits
  int32_t stride, ns, m;   // sample: one of every `stride` codes, ns in all, threshold at its m-th largest
  int32_t take_all;     // the list takes every code
  int32_t most;         // sampled codes above a threshold, at which the list is likely to overflow
  int32_t splits;       // (long rows) blocks that share the tiles of a group of 128 rows
  int32_t statblocks;
  const float* Ep;      // [V][PD]: the codebook itself where its rows start on 16 bytes, or a padded copy
  float* copy;          // where that is made, or null
  i32x4* Ef;            // long rows: [Vp/16][KS][3 limbs][64 lanes] fragments
                        // short rows: [Vp][2 N] pieces of 8 halves, the upper ones, then the lower ones
  i32x4* Es;            // the sample's codes, packed: long rows [ns/16][KS][64 lanes] upper limbs, short rows [ns][2 N]
  i32x4* Ew;            // short rows: Ef and Es of the halves of kWideScale
  i32x4* Ews;
  float* norms;         // [V]
  float* l1;            // [V]
  uint32_t* hash;       // (long rows) [V] of a code's numbers and their order
  int32_t* seen;        // (long rows) [2][1 << 32 - seen_shift] codes by their hash, in one place and in another
  int32_t* twin;        // (long rows) [V] a code that is the same, one for all of them
  int32_t seen_shift;
  float4* part;         // [kStatBlocks]: max norm, max |x|, max 1-norm, any NaN
  RowPlan* plan;        // [Vp]
  float* reach;         // [Vp] what the magnitudes of a row's products with any code add up to at most (long rows)
  int32_t* cnt;         // [V] entries of the row's list, or more than `cap` where it overflowed
  uint32_t* cand;       // [V][cap]
  int32_t* redo;        // [1 + V]: rows that take the exact path, their number first
  int32_t* neigh;       // [V][k]
};

struct Stats { float norm, mabs, l1, nan; };

// Four halves of a short row's upper (h) and lower (l) parts, dimensions d .. d + 3; what lies behind them in
// the piece of eight is zeroed by the lane that holds the row's last four.
template <typename F4>
__device__ __forceinline__ void put_halves(i32x4* base, int row, int n8, int d, F4 h, F4 l) {
  F4* hp = reinterpret_cast<F4*>(base + (int64_t)row * 2 * n8) + d / 4;
  F4* lp = reinterpret_cast<F4*>(base + (int64_t)row * 2 * n8 + n8) + d / 4;
  *hp = h;
  *lp = l;
}

// The four maxima over the stat kernel's blocks; every lane of the wave returns them.
__device__ __forceinline__ Stats reduce_stats(const KnnArgs& a, int lane) {
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < kStatBlocks / 64; ++i) {
    const float4 x = a.part[min(lane + 64 * i, a.statblocks - 1)];
    v[0] = fmaxf(v[0], x.x); v[1] = fmaxf(v[1], x.y); v[2] = fmaxf(v[2], x.z); v[3] = fmaxf(v[3], x.w);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {                             // (none is below zero)
#define LPP_MAX(ctrl, rows) v[q] = fmaxf(v[q], __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[q]), ctrl, rows, 0xf, false)))
    LPP_MAX(0x111, 0xf); LPP_MAX(0x112, 0xf); LPP_MAX(0x114, 0xf); LPP_MAX(0x118, 0xf);     // row_shr:1, 2, 4, 8
    LPP_MAX(0x142, 0xa); LPP_MAX(0x143, 0xc);               // row_bcast:15, 31
#undef LPP_MAX
    v[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[q]), 63));
  }
  return Stats{v[0], v[1], v[2], v[3]};
}

// The sample: of every `stride` consecutive codes (a power of two) one, at a place that a hash of the
// stratum picks, so that a codebook with an order of its own is sampled evenly.  Its number, or -1.
__device__ __forceinline__ int sample_slot(const KnnArgs& a, int code) {
  const int j = code / a.stride;
  const uint32_t off = (((uint32_t)j * 2654435761u) >> 15) & (uint32_t)(a.stride - 1);
  return j < a.ns && code == j * a.stride + (int)off ? j : -1;
}

// One number more in a lane's share of the hash of a code (no products, which issue at a quarter of the rate).
__device__ __forceinline__ uint32_t hash_in(uint32_t h, float x) {
  h ^= __float_as_uint(x);
  h += h << 10;
  return h ^ __builtin_amdgcn_alignbit(h, h, 6);
}
// The hash of a code held by G lanes: the last of them returns it.
template <int G>
__device__ __forceinline__ uint32_t hash_end(uint32_t h) {
  h = (h ^ h >> 15) * 2246822519u;
  h ^= h >> 13;
  h += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x128, 0xf, 0xf, false);       // row_ror:8, 4, 2, 1
  h += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x124, 0xf, 0xf, false);
  h += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x122, 0xf, 0xf, false);
  h += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x121, 0xf, 0xf, false);
  if (G == 64) {
    h += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x142, 0xa, 0xf, false);     // row_bcast:15 into rows 1 and 3
    h += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x143, 0xc, 0xf, false);     // row_bcast:31 into rows 2 and 3
  }
  return h;
}

// The two places of a code in `seen`; its copies are found unless other codes took both.  (One place, and a group of 64
// copies whose place another code took: 8192 x 256, k = 100 280 us instead of 232.  By the 1-norm instead of a hash, codes of one
// set of numbers with their signs turned shared a place: 8192 x 256, each four times, k = 1000 1.68 ms and now 0.43.)
__device__ __forceinline__ uint32_t seen_slot(const KnnArgs& a, uint32_t hash) { return hash >> a.seen_shift; }
__device__ __forceinline__ uint32_t other_slot(const KnnArgs& a, uint32_t hash) {
  return (1u << (32 - a.seen_shift)) + (hash * 2654435761u >> a.seen_shift);
}

// Over the G lanes of a row, without LDS; every lane returns it.
template <int G, typename F>
__device__ __forceinline__ float over_lanes(float x, F join) {
#define LPP_JOIN(ctrl, rows) x = join(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, rows, 0xf, false)))
  LPP_JOIN(0xB1, 0xf);                                      // quad_perm: one lane on, two lanes on
  LPP_JOIN(0x4E, 0xf);
  if (G >= 16) {
    LPP_JOIN(0x141, 0xf);                                   // row_half_mirror, row_mirror
    LPP_JOIN(0x140, 0xf);
  }
  if (G == 64) {
    LPP_JOIN(0x142, 0xa);                                   // row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3
    LPP_JOIN(0x143, 0xc);
    x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
  }
#undef LPP_JOIN
  return x;
}

// G lanes per row, 16 bytes per lane and step.  Bound by latency: the fewer rows one after the other the better, 256 blocks
// and sums over lanes without LDS.  (128 blocks, through LDS, and
// the copy made always: 8192 x 256 13.6 us and now 5.2, the build 187.6 and 178.4.)
template <int G>
__global__ __launch_bounds__(kStatThreads) void knn_stats_kernel(KnnArgs a) {
  constexpr int W = kStatThreads / 64;
  __shared__ float s_part[4][W];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = threadIdx.x % G;
  const bool vec = a.copy == nullptr;
  if (blockIdx.x == 0 && threadIdx.x == 0) a.redo[0] = 0;
  float mx[4] = {0.f, 0.f, 0.f, 0.f};
  // (short rows: zeros in the halves of the rows from V on, see CollectQuery)
  for (int row = blockIdx.x * (kStatThreads / G) + threadIdx.x / G; row < (G == 4 ? a.Vp : a.V); row += gridDim.x * (kStatThreads / G)) {
    const bool there = G != 4 || row < a.V;
    const float* src = a.E + (int64_t)row * a.D;
    float* dst = a.copy + (int64_t)row * a.PD;
    float ss = 0.f, sa = 0.f, mb = 0.f;
    uint32_t hash = (uint32_t)(sub + 1) * 2246822519u;
    // (short rows: whole pieces of eight halves, zero past the row)
    const int dend = G == 4 ? (a.D > 8 ? 16 : 8) : a.PD;
    for (int d = 4 * sub; d < dend; d += 4 * G) {
      float v[4];
      if (!there) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = 0.f;
      } else if (vec && d < a.D) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(src + d);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = x[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = d + e < a.D ? src[d + e] : 0.f;
      }
      if (a.copy && there && d < a.PD) *reinterpret_cast<f32x4*>(dst + d) = f32x4{v[0], v[1], v[2], v[3]};
      if (G == 4) {
        // scale x = h + l + rest: two halves of 11 bits each (rest: at most 2^-24 of it, or 2^-25).  Both scales:
        // which one holds is known when all rows have been here.
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        const int n8 = a.D > 8 ? 2 : 1;                     // pieces of 8 halves per part
        const int j = sample_slot(a, row);
#pragma unroll
        for (int wide = 0; wide < 2; ++wide) {
          f16x4 h, l;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = v[e] * (wide ? kWideScale : kHalfScale);
            h[e] = (_Float16)x;
            l[e] = (_Float16)(x - (float)h[e]);
          }
          if (j >= 0) put_halves(wide ? a.Ews : a.Es, j, n8, d, h, l);
#pragma unroll
          for (int e = 0; e < 4; ++e)                         // (see CollectQuery: NaN, and what the scale takes beyond the halves' range)
            if (!(fabsf((float)h[e]) < INFINITY)) { h[e] = (_Float16)0.f; l[e] = (_Float16)0.f; }
          put_halves(wide ? a.Ew : a.Ef, row, n8, d, h, l);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (G > 4) hash = hash_in(hash, v[e]);
        ss += v[e] * v[e];
        sa += fabsf(v[e]);
        mb = fmaxf(mb, fabsf(v[e]));
      }
    }
    const auto add = [](float x, float y) { return x + y; };
    const auto larger = [](float x, float y) { return fmaxf(x, y); };
    ss = over_lanes<G>(ss, add);
    sa = over_lanes<G>(sa, add);
    mb = over_lanes<G>(mb, larger);
    const float n = sqrtf(ss);
    if (there && sub == 0) { a.norms[row] = n; a.l1[row] = sa; }
    if (G > 4 && sub == 0) a.cnt[row] = 0;
    if (G > 4) hash = hash_end<G>(hash);
    if (G > 4 && sub == G - 1) a.hash[row] = hash;
    // (a row that holds a NaN has a NaN norm and takes no part in the maxima)
    const bool bad = !(n == n);
    mx[0] = fmaxf(mx[0], n);
    mx[1] = fmaxf(mx[1], bad ? 0.f : mb);
    mx[2] = fmaxf(mx[2], sa);
    mx[3] = fmaxf(mx[3], bad ? 1.f : 0.f);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int q = 0; q < 4; ++q) mx[q] = fmaxf(mx[q], __shfl_xor(mx[q], o));
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) s_part[q][wave] = mx[q];
  __syncthreads();
  if (threadIdx.x < 4) {
    const int q = threadIdx.x;
    float m = s_part[q][0];
#pragma unroll
    for (int w = 1; w < W; ++w) m = fmaxf(m, s_part[q][w]);
    reinterpret_cast<float*>(a.part + blockIdx.x)[q] = m;
  }
}

// Unit of the fixed-point image (as a double: q = round(x / unit) is then exact to half a unit).
__device__ __forceinline__ double limb_unit(float mabs) {
  return mabs > 0.f && mabs < INFINITY ? (double)mabs / (double)kLimbRange : 1.0;
}

// One lane per (tile of 16 codes, step of 64 dimensions, fragment lane): 16 dimensions of one code.
template <int KS>
__global__ __launch_bounds__(256) void knn_limb_kernel(KnnArgs a) {
  const int idx = blockIdx.x * 256 + threadIdx.x;            // (the grid covers Vp/16 * KS * 64 lanes exactly)
  const int lane = idx & 63, ks = (idx >> 6) % KS, tile = (idx >> 6) / KS;
  const int row = tile * 16 + (lane & 15), d0 = ks * 64 + (lane >> 4) * 16;
  const uint32_t hash = a.hash[min(row, a.V - 1)];
  const float l1 = a.l1[min(row, a.V - 1)];
  const Stats st = reduce_stats(a, threadIdx.x & 63);
  const double inv = 1.0 / limb_unit(st.mabs);
  const bool ok = row < a.V && a.norms[min(row, a.V - 1)] == a.norms[min(row, a.V - 1)];
  if (ks == 0 && lane < 16 && row < a.V && l1 > 0.f) {       // (any of the codes that share a place)
    a.seen[seen_slot(a, hash)] = row;
    a.seen[other_slot(a, hash)] = row;
  }
  uint32_t limb[3][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (ok && d0 + 4 * c < a.PD) x = *reinterpret_cast<const f32x4*>(a.Ep + (int64_t)row * a.PD + d0 + 4 * c);
    uint32_t wa = 0, wb = 0, wc = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double r = fmin(fmax((double)x[e] * inv, -(double)kLimbRange), (double)kLimbRange);
      const int q = (int)rint(r);
      const int lc = ((q + 128) & 255) - 128, q1 = (q - lc) >> 8;
      const int lb = ((q1 + 128) & 255) - 128, la = (q1 - lb) >> 8;      // |la| <= 127
      wa |= (uint32_t)(la & 255) << (8 * e);
      wb |= (uint32_t)(lb & 255) << (8 * e);
      wc |= (uint32_t)(lc & 255) << (8 * e);
    }
    limb[0][c] = wa; limb[1][c] = wb; limb[2][c] = wc;
  }
  i32x4* dst = a.Ef + ((int64_t)(tile * KS + ks) * 3) * 64 + lane;
#pragma unroll
  for (int l = 0; l < 3; ++l) dst[64 * l] = i32x4{(int)limb[l][0], (int)limb[l][1], (int)limb[l][2], (int)limb[l][3]};
  const int j = row < a.V ? sample_slot(a, row) : -1;
  if (j >= 0) a.Es[(int64_t)((j >> 4) * KS + ks) * 64 + (lane & 48) + (j & 15)] = dst[0];
}

// Short rows on the f16 matrix cores: x = h + l, and h h' + l h' + h l' of up to 8 N dimensions take N
// MFMA of 32 (16 cycles each and beside the vector instructions; the fp32 MFMA takes 32 cycles per 4
// dimensions and competes with them).  Slot g of the first MFMA: N = 1: h l h - of the code against
// h h l 0 of the query; N = 2: h0 h1 l0 l1 against h0 h1 h0 h1, and in the second h0 h1 - - against
// l0 l1 0 0 (- : any of the code's own numbers).
template <int N>
struct HalfOperand {
  f16x8 x[N];
  // (tile: the same for the wave; its 16 codes are there, whatever those past the end hold)
  __device__ __forceinline__ void load_code(const i32x4* tile, int l16, int g4) {
    const uint32_t row = (uint32_t)(l16 * 2 * N);
    x[0] = __builtin_bit_cast(f16x8, tile[row + (N == 1 ? (g4 == 1 ? 1 : 0) : g4)]);
    if (N == 2) x[N - 1] = __builtin_bit_cast(f16x8, tile[row + (g4 & 1)]);
  }
  __device__ __forceinline__ void load_query(const i32x4* row, int g4) {
    const i32x4 zero = {0, 0, 0, 0};
    if (N == 1) {
      x[0] = __builtin_bit_cast(f16x8, g4 == 3 ? zero : row[g4 == 2 ? 1 : 0]);
    } else {
      x[0] = __builtin_bit_cast(f16x8, row[g4 & 1]);
      x[N - 1] = __builtin_bit_cast(f16x8, g4 >= 2 ? zero : row[2 + g4]);
    }
  }
  __device__ __forceinline__ f32x4 times(const HalfOperand& q, f32x4 acc) const {
#pragma unroll
    for (int i = 0; i < N; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x[i], q.x[i], acc, 0, 0, 0);
    return acc;
  }
};

// The same for the collecting sweep, whose loads bring 64 bytes a cycle and compute unit whatever is in them: every piece of a
// code is loaded once, and a second MFMA takes the products with the query's lower parts.  N = 1: an operand holds the
// pieces of two tiles, h l of the one and h l of the other, against h h 0 0 and l 0 0 0 or 0 0 h h and 0 0 l 0; N = 2:
// h0 h1 l0 l1 against h0 h1 h0 h1 and l0 l1 0 0.  A code's numbers meet zeros in place of another's, and zero times infinity is
// NaN: every half has to be finite, also in the rows from V on and in a code that holds a NaN, whose other numbers may be as large as
// they like (it takes no part in the codebook's largest magnitude).  knn_stats puts zeros where one is not.  That changes nobody's
// similarity: a code that holds a NaN is left out when it is ranked, and of other codes such a number takes all rows to the exact path.
template <int N>
struct CollectQuery {
  f16x8 h[3 - N], l[3 - N];
  __device__ __forceinline__ void load(const i32x4* row, int g4) {
    const i32x4 zero = {0, 0, 0, 0};
    if (N == 1) {
      const i32x4 up = row[0], low = row[1];
#pragma unroll
      for (int t = 0; t < 3 - N; ++t) {
        h[t] = __builtin_bit_cast(f16x8, g4 >> 1 == t ? up : zero);
        l[t] = __builtin_bit_cast(f16x8, g4 == 2 * t ? low : zero);
      }
    } else {
      h[0] = __builtin_bit_cast(f16x8, row[g4 & 1]);
      l[0] = __builtin_bit_cast(f16x8, g4 >= 2 ? zero : row[2 + g4]);
    }
  }
  __device__ __forceinline__ f32x4 times(f16x8 code, int tile, f32x4 acc) const {
    const int t = N == 1 ? tile : 0;
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(code, h[t], acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(code, l[t], acc, 0, 0, 0);
  }
};

// Histogram of 16 NQ rows' similarities with the sample, the threshold bin of each row, and its plan.
// N: pieces of 8 dimensions (short rows, FIXED = false) or steps of 64 limbs (FIXED).  The
// histogram is laid out bin by bin with 16 rows side by side, so the 64 lanes of an LDS add,
// four per row, meet in at most a few banks: [bins][16] counts, 64 KB, two
// blocks per compute unit.  (With rows of bins one after the other the adds collide at random and a
// wave-wide add takes about 29 cycles.)  NQ = 2: 32 rows, a word counts for row l16 in its lower half and for row 16 + l16 in its upper
// one (a sample has fewer than 2 kSampleCodes codes).  What that halves: the sample's codes out of L2, which bound the
// kernel for long rows (8192 x 256: 28.5 -> 21.5 us, 7.5 of it not the sweep), and the turns of blocks at everything that is not
// the sweep (16384 x 8: 26 -> 21 us; 12.5 of 28 were not).
template <bool FIXED, int N, int NQ>
__global__ __launch_bounds__(kSampleThreads, FIXED && NQ == 2 && N >= 3 ? 4 : 8) void knn_sample_kernel(KnnArgs a) {
  extern __shared__ __align__(16) uint32_t s_hist[];      // [kSampleBins][16]
  constexpr int SEG = kSampleThreads / 16, SW = kSampleBins / SEG;   // segments of the bins, bins of each
  constexpr int R = 16 * NQ;                               // rows of the block
  __shared__ uint32_t s_seg[kSampleThreads / 64][16];      // counts of a wave's segments, per row
  __shared__ int s_top[R], s_upper[R], s_bin[R], s_fine[R], s_crowded[R + 1];   // [R]: any row
  constexpr int W = kSampleThreads / 64;
  static_assert(2 * kSampleCodes <= 65536, "two counts in a word");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = blockIdx.x * R;
  // (for the look at the rows' copies below, two to a wave: asked for now; 16 rows: by waves 1 .. 8)
  const int own = min(max(row0 + 2 * (NQ == 2 ? wave : wave - 1) + (lane >> 5), 0), a.V - 1);
  const uint32_t own_hash = FIXED ? a.hash[own] : 0u;
  const Stats st = reduce_stats(a, lane);
  const int seen1 = FIXED ? a.seen[seen_slot(a, own_hash)] : 0, seen2 = FIXED ? a.seen[other_slot(a, own_hash)] : 0;
  // lane: row l16 of each 16 for the sweep, row `lane` for the plan
  const int row = row0 + (lane & (R - 1)), rowc = min(row, a.V - 1);
  const float norm = a.norms[rowc], l1 = a.l1[rowc];
  const float top = norm * st.norm * 1.0001f;              // |similarity| stays below
  const bool wide = !FIXED && st.mabs * kHalfScale >= 65504.0f;
  const float hscale = wide ? kWideScale : kHalfScale;
  const double unit = FIXED ? limb_unit(st.mabs) : 1.0 / hscale;
  // one step of the histogram's argument: products of scaled halves, or of upper limbs (2^32 unit^2)
  const float to_sim = (float)(FIXED ? unit * unit * 4294967296.0 : unit * unit);
  // (far below 1e-30 the bound on the error would itself be rounded)
  const bool finite = top > 1e-30f && top < INFINITY && (FIXED || st.mabs * hscale < 65504.0f);

  if (!a.take_all) {
    if (tid < R) { s_top[tid] = 0; s_bin[tid] = 0; }
    if (tid <= R) s_crowded[tid] = 0;
    const int ntiles = (a.ns + 15) / 16;
    float per_bin[NQ], middle[NQ];
    bool fin[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const float mine = finite ? (kSampleBins / 2) * to_sim / top : 0.f;
      per_bin[n] = NQ == 1 ? mine : __shfl(mine, (lane & 15) + 16 * n);
      middle[n] = kSampleBins / 2;
      fin[n] = per_bin[n] != 0.f;
    }
    // (codes past the sample's end are not counted, nor is the row itself: where it is in the sample its own similarity,
    // often far above the others, would stretch the list's values over a range that holds nobody: 8192 x 256, k = 1000,
    // half the rows: buckets of 15 entries instead of 3)
    auto count = [&](float x0, float x1, float x2, float x3, int t, int n, int l16, int g4) {
      const float x[4] = {x0, x1, x2, x3};
      const uint32_t one = n ? 65536u : 1u;
      auto add = [&](float v) {
        const uint32_t bin = min((uint32_t)__builtin_fmaf(v, per_bin[n], middle[n]), kSampleBins - 1u);   // (negative, NaN: 0)
        atomicAdd(&s_hist[bin * 16 + l16], one);
      };
      const int own_tile = (row0 + 16 * n) / a.stride >> 4;   // (16 rows from a multiple of 16 on: one tile of the sample)
      if ((t + 1) * 16 <= a.ns && !(FIXED && t == own_tile)) {   // uniform
#pragma unroll
        for (int r = 0; r < 4; ++r) add(x[r]);
      } else {
        const int own = FIXED ? sample_slot(a, row0 + 16 * n + l16) : -1;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t * 16 + 4 * g4 + r < a.ns && t * 16 + 4 * g4 + r != own) add(x[r]);
      }
    };
    constexpr int U = FIXED && N >= 3 ? NQ : (N == 2 && (FIXED || NQ == 2) ? 2 : 4);
    auto sweep = [&](int tid) {
      const int l16 = tid & 15, g4 = (tid >> 4) & 3;
      auto clear = [&]() {
        for (int i = tid; i < kSampleBins * 4; i += kSampleThreads) reinterpret_cast<uint4*>(s_hist)[i] = make_uint4(0, 0, 0, 0);
        __syncthreads();
      };
      if constexpr (FIXED) {
        clear();
        i32x4 q[NQ][N];
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
          for (int ks = 0; ks < N; ++ks) q[n][ks] = a.Ef[((int64_t)((blockIdx.x * NQ + n) * N + ks) * 3) * 64 + (g4 * 16 + l16)];
        for (int t0 = wave; t0 < ntiles; t0 += W * U) {
          i32x4 f[U][N];
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int ks = 0; ks < N; ++ks) f[u][ks] = a.Es[(min(t0 + W * u, ntiles - 1) * N + ks) * 64 + (g4 * 16 + l16)];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            i32x4 acc[NQ];
#pragma unroll
            for (int n = 0; n < NQ; ++n) acc[n] = i32x4{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < N; ++ks)
#pragma unroll
              for (int n = 0; n < NQ; ++n) acc[n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[u][ks], q[n][ks], acc[n], 0, 0, 0);
            if (t0 + W * u < ntiles)
#pragma unroll
              for (int n = 0; n < NQ; ++n)
                count((float)acc[n][0], (float)acc[n][1], (float)acc[n][2], (float)acc[n][3], t0 + W * u, n, l16, g4);
          }
        }
      } else {
        const i32x4* const sampled = wide ? a.Ews : a.Es;
        HalfOperand<N> q[NQ], f[U];
        auto load = [&](int t0) {
#pragma unroll
          for (int u = 0; u < U; ++u) f[u].load_code(sampled + (int64_t)min(t0 + W * u, ntiles - 1) * (32 * N), l16, g4);
        };
#pragma unroll
        for (int n = 0; n < NQ; ++n)
          q[n].load_query((wide ? a.Ew : a.Ef) + (int64_t)min(row0 + 16 * n + l16, a.V - 1) * 2 * N, g4);
        clear();
        for (int t0 = wave; t0 < ntiles; t0 += W * U) {
          load(t0);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            f32x4 acc[NQ];
#pragma unroll
            for (int n = 0; n < NQ; ++n) acc[n] = f[u].times(q[n], f32x4{0.f, 0.f, 0.f, 0.f});
            if (t0 + W * u < ntiles)
#pragma unroll
              for (int n = 0; n < NQ; ++n) count(acc[n][0], acc[n][1], acc[n][2], acc[n][3], t0 + W * u, n, l16, g4);
          }
        }
      }
    };
    // thread (row, segment of bins): its count, then the segment the target-th largest lies in.  A wave
    // holds four segments of every row: sums over the waves go through LDS, inside a wave over lanes.  (Two rows' counts in
    // a word are added as they are.)
    auto search = [&](int target, int* s_found, bool first, int tid) {
      const int hr = tid & 15, seg = tid >> 4, g4 = seg & 3;
      auto part = [](uint32_t x, int n) { return (int)(NQ == 1 ? x : (n ? x >> 16 : x & 0xFFFFu)); };
      uint32_t local = 0;
      int high[NQ];
#pragma unroll
      for (int n = 0; n < NQ; ++n) high[n] = -1;
#pragma unroll
      for (int i = 0; i < SW; ++i) {
        const uint32_t c = s_hist[(seg * SW + i) * 16 + hr];
        local += c;
#pragma unroll
        for (int n = 0; n < NQ; ++n)
          if (part(c, n)) high[n] = SW * seg + i;
      }
      uint32_t above = 0;                                  // counts of the segments above mine
      {
        const uint32_t x1 = __shfl_down(local, 16), x2 = __shfl_down(local, 32), x3 = __shfl_down(local, 48);
        above = (g4 < 3 ? x1 : 0) + (g4 < 2 ? x2 : 0) + (g4 < 1 ? x3 : 0);
        if (g4 == 0) s_seg[wave][hr] = above + local;
      }
#pragma unroll
      for (int n = 0; n < NQ; ++n)
        if (first && high[n] >= 0) atomicMax(&s_top[hr + 16 * n], high[n]);
      __syncthreads();
      for (int w = wave + 1; w < W; ++w) above += s_seg[w][hr];
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        int over = part(above, n);
        if (over < target && target <= over + part(local, n)) {
          int i = SW - 1;
          for (;; --i) {
            over += part(s_hist[(seg * SW + i) * 16 + hr], n);
            if (i == 0 || over >= target) break;
          }
          s_found[hr + 16 * n] = SW * seg + i;
          // (bin 0 holds what lies below the range as well: no use looking closer)
          if (!FIXED && first && fin[n] && over > a.most && SW * seg + i > 0) s_crowded[hr + 16 * n] = s_crowded[R] = 1;
        }
      }
      __syncthreads();
    };
    sweep(tid);
    __syncthreads();
    search(a.m, s_bin, true, tid);
    // So many codes in the threshold's bin that some list would overflow (a few codes far longer than the others
    // stretch the bins, or a row has many near its largest): that bin once more, in as many parts.  The list's
    // values then end where its upper eighth begins, what lies above is ordered by keys (only of the rows that asked).  16384 x 8, k = 16, 100,
    // 1000, one code of length 300: 7.0, 7.1, 6.2 ms on the exact path -> 0.13, 0.16, 0.62; 16384 x 2: k = 16 3.2 ->
    // 0.16 ms.  (Long rows: their upper limbs would not tell the parts apart.)
    if (!FIXED && __builtin_amdgcn_readfirstlane(s_crowded[R])) {
      const int t = formed_anew(tid);                      // (nothing of it is kept in registers before)
      search(max(a.m / 8, 1), s_upper, false, t);
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        per_bin[n] *= kSampleBins;
        middle[n] = (float)(kSampleBins / 2 - s_bin[(t & 15) + 16 * n]) * kSampleBins;
      }
      sweep(t);
      __syncthreads();
      search(a.m, s_fine, false, t);
    }
  }
  // A code that is the same as this one, the same for all of them, or the code itself.  (seen holds what was written to
  // the place last, and rubbish where nothing was: what counts is that the numbers are the same.)
  // A row to 32 lanes; of 16 rows none to wave 0, which has the plans to make.  (To four lanes: 14.0 us, not 11.1, 1024 x 256, each code four times.)
  if (FIXED && (NQ == 2 || (wave >= 1 && wave <= 8))) {
    const int d = 4 * (lane & 31);
    auto holds = [&](int r) { return r >= 0 && r < a.V && a.hash[min(max(r, 0), a.V - 1)] == own_hash; };
    const bool first = holds(seen1), second = holds(seen2);
    const int r = first ? seen1 : seen2;
    bool same = (first || second) && r != own && a.l1[own] > 0.f;
    if (same) {
      const float* const x = a.Ep + (int64_t)own * a.PD;
      const float* const y = a.Ep + (int64_t)r * a.PD;
      i32x4 differ = {0, 0, 0, 0};
#pragma unroll
      for (int h = 0; h < 256; h += 128)
        if (d + h < a.PD) differ |= *reinterpret_cast<const i32x4*>(x + d + h) ^ *reinterpret_cast<const i32x4*>(y + d + h);
      same = (differ[0] | differ[1] | differ[2] | differ[3]) == 0;
    }
    const bool all_same = (uint32_t)(__ballot(same) >> (lane & 32)) == 0xFFFFFFFFu;
    if (d == 0) a.twin[own] = all_same ? r : own;           // (rows past the end: the last one's again)
  }
  if (tid >= R) return;

  // ---- the row's plan (lane = row)
  RowPlan p;
  const int vb = a.vmask_bits;
  const uint32_t qmax = (1u << vb) - 2u;
  const bool all = a.take_all || !finite;
  float thr, hi;
  if (all) {
    thr = finite ? -top : 0.f;
    hi = finite ? top : 1.f;
  } else {
    // (bin 0 also holds what lies below the range)
    const float width = top / (kSampleBins / 2);
    const float fine = !FIXED && s_crowded[tid] ? (float)s_fine[tid] / kSampleBins : 0.f;
    thr = s_bin[tid] > 0 ? ((float)(s_bin[tid] - kSampleBins / 2) + fine) * width : -top;
    hi = (float)((!FIXED && s_crowded[tid] ? s_upper[tid] : s_top[tid]) + 1 - kSampleBins / 2) * width;
    hi = fminf(hi + 0.125f * (hi - thr), top);
    hi = fmaxf(hi, thr + 0.25f * width);
  }
  // rounding bound of an approximate similarity
  float e;
  if (FIXED) {
    const double u = unit;
    const double trunc = 3.0 * 16777216.0 * u * u;         // cut low parts: below three units of the value kept
    e = (float)(0.5005 * u * ((double)l1 + (double)st.l1) * 1.001 + a.D * u * u + trunc);
  } else {
    // up to 32 N products that are not zero on top of the threshold, each sum rounded by 2^-23; l l' and what the halves leave of
    // each number: 3 2^-22, or 2^-25 of the scaled number
    e = (float)(32 * N + 6) * 1.1920929e-07f * (norm * st.norm + fabsf(thr)) * 1.001f + 7.2e-07f * norm * st.norm +
        2.9802322e-08f / hscale * (l1 + st.l1) * 1.001f + 1e-30f;
  }
  e += norm * st.norm * 1e-9f;
  float range = hi - thr;
  // below the bin's edge by more than the test at the end asks of the (k-1)-th entry
  const float slack = 2.2f * e + (6.0f + 2.0f * (float)list_rounding(qmax)) * range / (float)qmax;
  thr -= slack;
  range += slack;
  // A row that holds a NaN, or only zeros beside a codebook of finite numbers (a code that was never used): every
  // similarity is the same, the lowest codes are its neighbours.  (On the exact path a wave took 0.8 to 9 ms for
  // such a row.  One NaN: 987 -> 137 us at 16384 x 8, k = 100, 9692 -> 218 us at 8192 x 256; a twentieth of zeros:
  // 1518 -> 134 us and 11.8 ms -> 212 us.)
  const bool flat = norm != norm || (l1 == 0.f && st.norm < INFINITY && !(st.nan > 0.f));
  p.flags = (all ? kAll : 0) | (st.nan > 0.f ? kAnyNan : 0) | (finite ? 0 : kNoList) | (flat ? kFlat : 0) |
            (wide ? kWide : 0);
  const double uu = FIXED ? unit * unit * 16777216.0 : unit * unit;      // real value of one unit of d
  p.a = (float)((double)qmax / ((double)range / uu));
  if (FIXED) p.thr_u = (int)fmin(fmax(floor((double)thr / uu), -1073741824.0), 1073741823.0);
  else p.thr = (float)((double)thr / uu);
  p.E = list_margin(e, range, qmax);
  if (row >= a.V || !finite) {                              // nothing passes
    p.a = 0.f;
    if (FIXED) p.thr_u = 1 << 30;
    else p.thr = INFINITY;
  }
  if (!(e < INFINITY)) p.E = 1 << 30;
  a.plan[row] = p;
  if (FIXED) a.reach[row] = l1 * st.mabs;                   // (not the norms: squares of small numbers vanish in them)
}

// Groups of 128 codes whose tiles a group's blocks take: itself and those up to half way round; of two that lie opposite
// the first.  Tiles of block `split` of `splits`.
__host__ __device__ inline int collect_tiles(int groups, int group, int split, int splits) {
  const int tiles = 8 * (groups % 2 ? groups / 2 + 1 : groups / 2 + (group < groups / 2 ? 1 : 0));
  return split < tiles ? (tiles - split + splits - 1) / splits : 0;
}

// What both collecting kernels do with the similarities they form: a lane holds four of one row per
// code tile, less the row's threshold (which the sums start from).  It parks them in LDS as they are
// and shifts their sign bits into a mask, one instruction each.  After a window of tiles the lanes take the clear bits
// of their masks and write the list words.  (With one LDS write per similarity, to a ring that only moved on where a
// similarity passed, the kernel was bound by issuing those writes.)
__device__ __forceinline__ uint32_t shift_in_sign(uint32_t mask, int d) { return __builtin_amdgcn_alignbit(mask, (uint32_t)d, 31); }

// mask: bit 31 - s set where similarity s of the window passes; word(s): its list word.  The lane's words go to cand
// from `at` on, which is in the list (a list that overflows is not used, nor written to).
// A word at a time: a store's lanes lie in as many places as there are lanes, which take the address unit a cycle or
// more each, 21 us of 79 at 16384 x 8, k = 1000.  One where their number is odd, then two, then four at a time: 4 us.
template <typename Word>
__device__ __forceinline__ void emit_window(uint32_t* cand, uint32_t at, uint32_t mask, Word word) {
  typedef uint32_t words2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef uint32_t words4 __attribute__((ext_vector_type(4), aligned(4)));
  auto take = [&]() {
    const uint32_t s = __builtin_clz(mask);
    mask &= ~(0x80000000u >> s);
    return word(s);
  };
  const int n = __popc(mask);
  if (n & 1) cand[at++] = take();
  if (n & 2) {
    const uint32_t x = take(), y = take();
    *reinterpret_cast<words2*>(cand + at) = words2{x, y};
    at += 2;
  }
  while (__any(mask != 0u)) {
    if (mask != 0u) {
      const uint32_t x = take(), y = take(), z = take(), w = take();
      *reinterpret_cast<words4*>(cand + at) = words4{x, y, z, w};
      at += 4;
    }
  }
}

// Short rows: a block owns 16 queries, its waves (as many as fill the chip) take windows of 128 codes in turn, eight
// MFMA tiles.  Which code a tile's row is, is free: lane (l16, g4) gets the similarities of the 32 consecutive codes from
// 32 g4 on, so that slot s of its window is code s, parked at [s][lane] (no two lanes of a read in one bank), and an
// entry's code, its place in LDS and its list word are an instruction or two each.  (Tiles of 16 consecutive codes: 17
// vector instructions an entry instead of 14; 16384 x 8, k = 1000: 79 -> 77 us, 58 with what emit_window does.)
constexpr int kCollectMaxWaves = 16;
constexpr int kWindowCodes = 128;
template <int N>
__global__ __launch_bounds__(kCollectMaxWaves * 64) void knn_collect_f16_kernel(KnnArgs a) {
  constexpr int T = kWindowCodes / 16;                     // tiles per window: 32 similarities a lane, 32 bits
  extern __shared__ __align__(16) uint32_t s_park[];       // [wave][32][64 lanes]
  __shared__ int s_cnt[16];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int row = blockIdx.x * 16 + l16, rowc = min(row, a.V - 1);
  const RowPlan p = a.plan[row];
  const int windows = a.Vp / kWindowCodes;                 // (rows V .. Vp - 1 are there and hold zeros, see CollectQuery)
  const float c0 = -p.thr;
  const i32x4* const Ef = __builtin_amdgcn_readfirstlane(p.flags) & kWide ? a.Ew : a.Ef;
  CollectQuery<N> q;
  q.load(Ef + (int64_t)rowc * 2 * N, g4);
  if (threadIdx.x < 16) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  uint32_t* const parked = s_park + wave * (T * 256) + lane;
  const uint32_t list = (uint32_t)rowc * (uint32_t)a.cap, qmax = (1u << a.vmask_bits) - 2u;
  const int step = blockDim.x >> 6, room = row < a.V ? a.cap : 0;
  // (N = 1: tiles in pairs, the second one's pieces in the upper 32 lanes)
  const i32x4* const lane_row = Ef + (32 * (l16 >> 2) + (l16 & 3)) * 2 * N + (N == 1 ? 8 * (g4 >> 1) + (g4 & 1) : g4);
  constexpr int F = T / 2 * N;                             // pieces per lane and window
  auto load = [&](f16x8 (&f)[F], int w) {                  // (past the end: the last window again, not used)
    const i32x4* const first = lane_row + (int64_t)min(w, windows - 1) * (kWindowCodes * 2 * N);
#pragma unroll
    for (int u = 0; u < F; ++u) f[u] = __builtin_bit_cast(f16x8, first[u * 16]);
  };
  f16x8 f[F], next[F];
  load(f, wave);
  for (int w = wave; w < windows; w += step) {
    load(next, w + step);
    uint32_t fail = 0;
#pragma unroll
    for (int h = 0; h < T; h += 4) {
      f32x4 acc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = q.times(f[N == 1 ? (h + u) / 2 : h + u], u & 1, f32x4{c0, c0, c0, c0});
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          parked[((h + u) * 4 + r) * 64] = __float_as_uint(acc[u][r]);
          fail = shift_in_sign(fail, __float_as_int(acc[u][r]));
        }
    }
    const int code0 = w * kWindowCodes + 32 * g4;
    uint32_t mask = ~fail;                                 // (codes past the end are not there)
    if (w == windows - 1) mask &= code0 + 32 <= a.V ? 0xFFFFFFFFu : (code0 < a.V ? ~(0xFFFFFFFFu >> (a.V - code0)) : 0u);
    // (the next window's pieces have to be here before the list words are written: loads and stores are counted together,
    // and a wait behind the stores, whose number differs, would be for all of them)
#pragma unroll
    for (int u = 0; u < F; ++u) {
      f[u] = next[u];
      asm volatile("" : "+v"(f[u]));
    }
    const int n = __popc(mask);
    const int base = n > 0 ? atomicAdd(&s_cnt[l16], n) : 0;
    emit_window(a.cand, list + (uint32_t)base, base + n > room ? 0u : mask,
                [&](uint32_t s) { return (list_value(__uint_as_float(parked[s * 64]), p.a, qmax) << a.ib) | (code0 + s); });
  }
  __syncthreads();
  if (threadIdx.x < 16 && blockIdx.x * 16 + threadIdx.x < a.V) a.cnt[blockIdx.x * 16 + threadIdx.x] = s_cnt[threadIdx.x];
}

// Long rows, fixed point: a wave owns 32 queries (two B operands, held in registers with all their
// limbs), a block's four waves 128.  Code tiles come through LDS, fragment by fragment as they lie
// in memory, one copy for the four waves (each limb fragment read feeds 32 queries), the next two
// chunks' loads in flight while one is worked on.  Two blocks per compute unit.
// The sums are the same whichever of two codes is the query, so each pair of groups of 128 codes is taken once: a group's
// blocks take the groups up to half way round from it (their tiles dealt to `splits` blocks), and a window's similarities,
// parked in LDS, are looked at a second time with a lane per code, 32 queries each, for the lists of the codes.
// The row's list is one, whoever adds to it: a wave asks for its places with an add in memory and has them when the
// products of the next tile are done; only then does it write the window's words.
// (Every pair from both sides, a list in segments, one per block that adds to it: the kernel 115 us at 8192 x 256,
// k = 1000, 78 of them its products alone, and now 77; the build 236 -> 191, 16384 x 256 696 -> 533, 4096 x 64, k = 300
// 57.9 -> 51.3, 1024 x 256, k = 100 38.0 -> 36.6.)
// Bound by the matrix cores, whose rate for 8-bit numbers the card's power limits (products of random numbers alone take
// 1.35 times what they would at 2.4 GHz, of numbers below 16 1.14 times), then by the windows' masks and words.
template <int KS>
__global__ __launch_bounds__(kCollectWaves * 64, 2) void knn_collect_i8_kernel(KnnArgs a) {
  constexpr int T = 4;                                     // tiles per window: 16 similarities per row and lane
  constexpr int CT = KS == 1 ? 4 : (KS == 2 ? 2 : 1);      // code tiles per chunk
  constexpr int TQ = KS * 3 * 64;                          // 16-byte pieces per tile
  constexpr int CQ = CT * TQ;                              // ... per chunk
  constexpr int NTHR = kCollectWaves * 64;
  static_assert(CQ % 64 == 0 && T % CT == 0, "chunks end with windows");
  constexpr int PER = (CQ + NTHR - 1) / NTHR;
  __shared__ i32x4 s_code[2][CQ];
  __shared__ i32x4 s_park[kCollectWaves][2][T * 64];       // [query tile][code tile][lane]: the lane's four codes
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int group = blockIdx.x / a.splits, split = blockIdx.x - group * a.splits;
  const int qtile = group * (kCollectWaves * 2) + wave * 2;
  const int ntiles = (a.V + 15) >> 4, alltiles = a.Vp >> 4;
  const uint32_t qmax = (1u << a.vmask_bits) - 2u;
  const i32x4* const Ef = a.Ef;
  int thr[2];
  float scale[2];
  i32x4 q[2][KS][3];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const RowPlan p = a.plan[(qtile + n) * 16 + l16];      // (rows past V: nothing passes)
    thr[n] = p.thr_u; scale[n] = p.a;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int l = 0; l < 3; ++l) q[n][ks][l] = Ef[((int64_t)((qtile + n) * KS + ks) * 3 + l) * 64 + lane];
  }
  // the group's tiles: its own eight, then those of the groups after it, half way round; of two groups that lie opposite
  // the first takes the pair.  This block's: split + i splits, i = 0 .. own - 1; chunk c holds i = c CT ..
  const int own = collect_tiles(a.Vp >> 7, group, split, a.splits);
  auto tile_at = [&](int i) {
    const int t = group * 8 + split + i * a.splits;
    return t < alltiles ? t : t - alltiles;
  };
  // two chunks' loads are in flight while a third is worked on (past the end: the last tile again, not used)
  struct Chunk { i32x4 x[PER]; };
  auto fetch = [&](int c) {
    Chunk k;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int o = min(tid + i * NTHR, CQ - 1);
      const int t = tile_at(min(c * CT + o / TQ, own - 1));
      k.x[i] = Ef[(int64_t)t * TQ + o % TQ];
    }
    return k;
  };
  auto park = [&](const Chunk& k, int b) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (CQ % NTHR == 0 || tid + i * NTHR < CQ) s_code[b][tid + i * NTHR] = k.x[i];
  };
  uint32_t fail[2] = {0, 0};
  // what a window leaves to be written
  struct Window {
    uint32_t rows[2], codes;                               // masks: a query's codes, a code's queries
    int before[2];                                         // entries of the row in the lanes before this one (of four)
    int at_row, at_code;                                   // places: lane 16 n + l16 holds row l16's of tile n; a code's own lane
    uint32_t code0;                                        // first code of the lane, without the turn round the end
    int code, thr;                                         // the code as a row, its plan
    float scale;
  } win;
  const int* const parked = reinterpret_cast<const int*>(s_park[wave]);
  // The lane's code in a window: tile lane >> 4, code lane & 15 of it, which lane group (lane >> 2) & 3 holds as its number
  // lane & 3.  Step s of the second look: query tile s >> 4, query (s & 15) ^ (lane >> 2), so that a read's lanes lie in 64 banks.
  const int turn = lane >> 2;
  const int* const column = parked + turn * 64 + (lane & 3);
  auto emit = [&]() {
    const uint32_t tile_step = (uint32_t)(16 * a.splits);
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int base = __shfl(win.at_row, 16 * n + l16) + win.before[n];
      const int row = min((qtile + n) * 16 + l16, a.V - 1);
      const int* const mine = parked + n * (T * 256) + lane * 4;
      emit_window(a.cand, (uint32_t)row * (uint32_t)a.cap + (uint32_t)base, base + __popc(win.rows[n]) <= a.cap ? win.rows[n] : 0u,
                  [&](uint32_t s) {
                    const uint32_t hi = s >> 2, lo = s & 3, t = __umul24(hi, tile_step) + win.code0;
                    return (list_value((float)(mine[hi * 256 + lo] - thr[n]), scale[n], qmax) << a.ib) | min(t, t - (uint32_t)a.Vp) | lo;
                  });
    }
    emit_window(a.cand, (uint32_t)win.code * (uint32_t)a.cap + (uint32_t)win.at_code,
                win.at_code + __popc(win.codes) <= a.cap ? win.codes : 0u, [&](uint32_t s) {
                  const uint32_t x = (s ^ (uint32_t)turn) & 15u, n = s >> 4;
                  return (list_value((float)(column[n * (T * 256) + x * 4] - win.thr), win.scale, qmax) << a.ib) |
                         ((uint32_t)(qtile * 16) + n * 16 + x);
                });
  };
  // the window that ends with the block's tile number i - 1: its masks, and its places are asked for
  auto close = [&](int i) {
    const int i0 = (i - 1) / T * T, have = i - i0;
    int total[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      // the four lanes of a row put their entries one after the other
      win.rows[n] = ~fail[n] << (32 - 4 * have);
      fail[n] = 0;
      const int cnt = __popc(win.rows[n]);
      const int c1 = __shfl(cnt, l16), c2 = __shfl(cnt, l16 + 16), c3 = __shfl(cnt, l16 + 32), c4 = __shfl(cnt, l16 + 48);
      win.before[n] = (g4 > 0 ? c1 : 0) + (g4 > 1 ? c2 : 0) + (g4 > 2 ? c3 : 0);
      total[n] = c1 + c2 + c3 + c4;
    }
    win.code0 = (uint32_t)((group * 8 + split + i0 * a.splits) * 16 + 4 * g4);
    const int mine = g4 == 0 ? total[0] : (g4 == 1 ? total[1] : 0);
    win.at_row = 0;
    if (mine > 0) win.at_row = __hip_atomic_fetch_add(a.cnt + (qtile * 16 + lane), mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the same similarities for the codes' lists (a group with itself has them in both its halves)
    const int it = i0 + (lane >> 4);
    const bool there = it < i && split + it * a.splits >= 8;
    win.codes = 0;
    if (split + (i - 1) * a.splits >= 8) {                 // uniform
      uint32_t miss = 0;
#pragma unroll
      for (int s = 0; s < 32; ++s)
        miss = shift_in_sign(miss, column[(s >> 4) * (T * 256) + (((s & 15) ^ turn) * 4)] - win.thr);
      uint32_t m = ~miss;
      if ((qtile + 2) * 16 > a.V) {                        // uniform: rows past the end are in nobody's list
        const int last = a.V - qtile * 16;
#pragma unroll 1
        for (int s = 0; s < 32; ++s)
          if ((s & 16) + ((s & 15) ^ turn) >= last) m &= ~(0x80000000u >> s);
      }
      win.codes = there ? m : 0u;
    }
    const int cnt = __popc(win.codes);
    win.at_code = 0;
    if (cnt > 0) win.at_code = __hip_atomic_fetch_add(a.cnt + win.code, cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  Chunk n0, n1;
  bool full = false;                                       // uniform: a window waits to be written
  auto tile_work = [&](const i32x4* tile, int i) {         // i: the block's tile number
    i32x4 aa[2], ab[2], bb[2], bc[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) aa[n] = ab[n] = bb[n] = bc[n] = i32x4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const i32x4 fa = tile[(ks * 3 + 0) * 64], fb = tile[(ks * 3 + 1) * 64], fc = tile[(ks * 3 + 2) * 64];
      // (products that add into the same sum are kept apart, so that none waits for the one before it)
#define LPP_LIMB(sum, f, l)                                                                    \
      sum[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f, q[0][ks][l], sum[0], 0, 0, 0);         \
      sum[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f, q[1][ks][l], sum[1], 0, 0, 0)
      LPP_LIMB(aa, fa, 0);
      LPP_LIMB(ab, fa, 1);
      LPP_LIMB(bb, fa, 2);
      LPP_LIMB(bc, fb, 2);
      LPP_LIMB(ab, fb, 0);
      LPP_LIMB(bb, fb, 1);
      LPP_LIMB(bc, fc, 1);
      LPP_LIMB(bb, fc, 0);
#undef LPP_LIMB
    }
    if (i % T == 0) {                                      // uniform
      if (full) {
        // (the chunks asked for have to be here before the list words are written: loads and stores are counted together,
        // and a wait behind the stores, whose number differs, would be for all of them)
#pragma unroll
        for (int x = 0; x < PER; ++x) asm volatile("" : "+v"(n0.x[x]), "+v"(n1.x[x]));
        emit();
      }
      win.code = tile_at(min(i + (lane >> 4), own - 1)) * 16 + l16;
      const RowPlan p = a.plan[win.code];
      win.thr = p.thr_u;
      win.scale = p.a;
    }
    const bool past = tile_at(i) >= ntiles;                // uniform: no codes there
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      i32x4 d;                                             // the similarity, in units of 2^24 unit^2 (each below 2^30, and so are the thresholds)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d[r] = (aa[n][r] << 8) + ab[n][r] + ((bb[n][r] + (bc[n][r] >> 8)) >> 8);
        fail[n] = shift_in_sign(fail[n], d[r] - thr[n]);
      }
      if (past) fail[n] |= 15u;
      s_park[wave][n][(i % T) * 64 + lane] = d;
    }
    full = (i + 1) % T == 0 || i + 1 == own;
    if (full) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");           // (the other lanes' similarities are read)
      __builtin_amdgcn_wave_barrier();
      close(i + 1);
    }
  };
  if (own == 0) return;                                    // uniform over the block
  n0 = fetch(0);
  n1 = fetch(1);
  auto work = [&](int c, int b) {
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      if (c * CT + j >= own) break;                        // uniform
      tile_work(s_code[b] + j * TQ + lane, c * CT + j);
    }
  };
  park(n0, 0);
  __syncthreads();
  for (int c = 0; c * CT < own; c += 2) {
    n0 = fetch(c + 2);
    work(c, 0);
    park(n1, 1);
    __syncthreads();
    if ((c + 1) * CT >= own) break;                        // uniform
    n1 = fetch(c + 3);
    work(c + 1, 1);
    park(n0, 0);
    __syncthreads();
  }
  emit();                                                  // (the last window ends with the block's last tile)
}

// ------------------------------------------------------------------------------------------ ranking

// A key as an integer of the same order.  NaN comes last, behind -inf: a code that holds one is nobody's
// neighbour while there are others, on every path.
__device__ __forceinline__ uint64_t orderable(double x) {
  if (x != x) return 1ull;
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// The codebook as the exact keys read it.  quads: rows start on 16 bytes and are padded with zeros to
// whole groups of four (a product of zeros leaves the chain as it is: it starts at +0 and can
// never be -0).
struct Rows {
  const float* p;
  int32_t pitch, D;
  bool quads;
  const int32_t* twin;                                      // (long rows) codes that are the same have the same here
};

// exact key of the pair (row i held in LDS as doubles, code j): float64 FMA chain in index order
__device__ __forceinline__ uint64_t exact_key(const double* ei, const Rows& R, int j) {
  const float* ej = R.p + (int64_t)j * R.pitch;
  double acc = 0.0;
  if (R.quads) {
    for (int t = 0; t < R.D; t += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(ej + t);
      const f64x2 e0 = *reinterpret_cast<const f64x2*>(ei + t), e1 = *reinterpret_cast<const f64x2*>(ei + t + 2);
      acc = __builtin_fma(e0[0], (double)v[0], acc);
      acc = __builtin_fma(e0[1], (double)v[1], acc);
      acc = __builtin_fma(e1[0], (double)v[2], acc);
      acc = __builtin_fma(e1[1], (double)v[3], acc);
    }
  } else {
    for (int t = 0; t < R.D; ++t) acc = __builtin_fma(ei[t], (double)ej[t], acc);
  }
  return orderable(acc);
}

// exact_key of U codes side by side, 64 bytes of each at a time: their chains do not wait for each other's loads.
template <int U>
__device__ __forceinline__ void exact_keys(const double* ei, const Rows& R, const int (&j)[U], uint64_t (&K)[U]) {
  if (!R.quads) {
#pragma unroll
    for (int u = 0; u < U; ++u) K[u] = exact_key(ei, R, j[u]);
    return;
  }
  double acc[U] = {};
  const float* ej[U];
#pragma unroll
  for (int u = 0; u < U; ++u) ej[u] = R.p + (int64_t)j[u] * R.pitch;
  for (int t0 = 0; t0 < R.D; t0 += 16) {
    f32x4 v[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (t0 + 4 * c < R.D) v[u][c] = *reinterpret_cast<const f32x4*>(ej[u] + t0 + 4 * c);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (t0 + 4 * c < R.D) {
        const f64x2 e0 = *reinterpret_cast<const f64x2*>(ei + t0 + 4 * c), e1 = *reinterpret_cast<const f64x2*>(ei + t0 + 4 * c + 2);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          acc[u] = __builtin_fma(e0[0], (double)v[u][c][0], acc[u]);
          acc[u] = __builtin_fma(e0[1], (double)v[u][c][1], acc[u]);
          acc[u] = __builtin_fma(e1[0], (double)v[u][c][2], acc[u]);
          acc[u] = __builtin_fma(e1[1], (double)v[u][c][3], acc[u]);
        }
      }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) K[u] = orderable(acc[u]);
}

__device__ __forceinline__ double key_value(uint64_t K) {
  const uint64_t u = (K >> 63) ? (K & 0x7FFFFFFFFFFFFFFFull) : ~K;
  return __longlong_as_double((long long)u);
}

// Sum over the 16 lanes of a DPP row; all of them return it.
__device__ __forceinline__ double add_over_16(double x) {
#define LPP_ROR(n)                                                                                                  \
  {                                                                                                                 \
    const uint64_t b = (uint64_t)__double_as_longlong(x);                                                           \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + n, 0xf, 0xf, false);       \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x120 + n, 0xf, 0xf, false); \
    x += __longlong_as_double((long long)((uint64_t)hi << 32 | lo));                                                \
  }
  LPP_ROR(8) LPP_ROR(4) LPP_ROR(2) LPP_ROR(1)
#undef LPP_ROR
  return x;
}

// (key desc, idx asc) "a goes before b"
__device__ __forceinline__ bool before(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return ka > kb || (ka == kb && ia < ib);
}

// Sum of one int per thread before this one, over a block of NTHR threads, and the total.
template <int NTHR>
__device__ __forceinline__ int block_exclusive(int v, int* s_w, int tid, int& total) {
  const int lane = tid & 63, wv = tid >> 6;
  int incl = v;
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, false);
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, false);
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, false);
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  if (lane == 63) s_w[wv] = incl;
  __syncthreads();
  int base = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < NTHR / 64; ++w) {
    if (w < wv) base += s_w[w];
    total += s_w[w];
  }
  return base + incl - v;
}

// LDS of the ranking, in 4-byte words: the row as doubles [PD], then buckets [NB] and the entries by
// bucket [P] (later the exact keys: NB >= P), the sorted entries [P], the list of those that need
// their keys [P / 2 words].  P: list capacity rounded up; NB: buckets, a power of two.
struct RankShape { int32_t P, lognb; };

// One row: w[] are the thread's entries -- list words inverted, so that the nearest comes first in ascending
// order: inverted value over inverted index -- `on` bit u set where w[u] is one; have: entries of the block, filled up round
// by round.
// Sorts them by value, orders what E leaves open by exact keys, writes the first kk codes to
// out[1..].  False: the list does not prove its first kk entries (out may be written all the same).
// Bound by LDS and vector instructions per entry, so each stage touches an entry once (and a round of entries that the
// list does not have is skipped; the buckets' counts stay in registers over the scan: 16384 x 8, k = 1000, the build
// 182 -> 178 us; k = 300: 139 -> 133): an LDS add that gives the
// place in the bucket, one read of the bucket's start, one write by bucket; entries more than E
// below the bucket of the kk-th are left out from there on.  The buckets hold a few entries each: a wave takes 64
// pairs in bucket order, 8 entries on either side shared with its neighbours, and eight rounds of
// odd-even transposition (inside the pairs, across the lanes) put them in order; what is next to what is then
// known in registers.
// (An entry more than E below the kk-th value has kk entries before it for certain, and so has one that is
// only before it by its key: neither can move anything among the first kk.)
template <int NTHR, int EPT, bool STAGED>
__device__ bool rank_row(const uint32_t (&w)[EPT], uint32_t on, int have, int ib, int vb, int E, bool all, int kk, const Rows& R,
                         float reach, RankShape sh, unsigned char* smem, int* s_w, int32_t* out, int tid) {
  const int NB = 1 << sh.lognb;
  double* eid = reinterpret_cast<double*>(smem);
  uint32_t* bucket = reinterpret_cast<uint32_t*>(eid + ((R.D + 3) & ~3));
  uint32_t* scat = bucket + NB;
  uint32_t* sorted = scat + sh.P;
  uint16_t* todo = reinterpret_cast<uint16_t*>(sorted + sh.P);
  uint64_t* key = reinterpret_cast<uint64_t*>(bucket);
  const int drop = 32 - min(sh.lognb, vb);                  // bucket number: the value's upper bits
  const uint32_t mask = (1u << ib) - 1u;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  enum { kTodo = 16, kKept, kLast, kCrowded, kFollow };
  constexpr int SIDE = 8;                                   // largest bucket the transposition rounds sort

  for (int i = tid; i < NB / 4; i += NTHR) reinterpret_cast<uint4*>(bucket)[i] = make_uint4(0, 0, 0, 0);
  if (tid == 0) { s_w[kTodo] = 0; s_w[kKept] = 0; s_w[kCrowded] = 0; }
  if (STAGED && tid == 0) s_w[kFollow] = 0;
  __shared__ uint32_t s_same[STAGED ? NTHR * EPT / 32 : 1];  // (long rows) bit p: sorted entry p is the same code as the one before it
  if (STAGED)
    for (int i = tid; i < NTHR * EPT / 32; i += NTHR) s_same[i] = 0;
  __syncthreads();
  uint32_t pos[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u)
    if (u * NTHR < have && ((on >> u) & 1u)) pos[u] = atomicAdd(&bucket[w[u] >> drop], 1u);
  __syncthreads();
  int n;
  {
    const int per = NB / NTHR;                              // four or eight, which stay in registers
    uint4 c[2];
    c[0] = *reinterpret_cast<const uint4*>(bucket + tid * per);
    c[1] = per == 8 ? *reinterpret_cast<const uint4*>(bucket + tid * per + 4) : make_uint4(0, 0, 0, 0);
    const int local = (int)(c[0].x + c[0].y + c[0].z + c[0].w + c[1].x + c[1].y + c[1].z + c[1].w);
    const uint32_t most = max(max(max(c[0].x, c[0].y), max(c[0].z, c[0].w)), max(max(c[1].x, c[1].y), max(c[1].z, c[1].w)));
    uint32_t run = (uint32_t)block_exclusive<NTHR>(local, s_w, tid, n);
    if (n < kk) return false;                               // uniform
    // (buckets behind the kk-th entry's play no part, however full)
    if ((int)run < kk && most > (uint32_t)SIDE) s_w[kCrowded] = 1;
    const bool last = (int)run < kk && (int)run + local >= kk;      // the kk-th entry lies in one of my buckets
    uint4 st[2];                                            // start | size << 16
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      st[h].x = run; st[h].y = st[h].x + c[h].x; st[h].z = st[h].y + c[h].y; st[h].w = st[h].z + c[h].z; run = st[h].w + c[h].w;
      if (last) {
        const int at = tid * per + 4 * h, k0 = kk - 1;      // (the bucket it lies in: the last that starts at or before it)
        if ((int)st[h].x <= k0 && (int)run > k0) s_w[kLast] = at + ((int)st[h].y <= k0) + ((int)st[h].z <= k0) + ((int)st[h].w <= k0);
      }
    }
    *reinterpret_cast<uint4*>(bucket + tid * per) =
        make_uint4(st[0].x | c[0].x << 16, st[0].y | c[0].y << 16, st[0].z | c[0].z << 16, st[0].w | c[0].w << 16);
    if (per == 8)
      *reinterpret_cast<uint4*>(bucket + tid * per + 4) =
          make_uint4(st[1].x | c[1].x << 16, st[1].y | c[1].y << 16, st[1].z | c[1].z << 16, st[1].w | c[1].w << 16);
  }
  __syncthreads();
  // whole buckets, up to the one that holds the last value of the kk-th entry's bucket plus E
  uint32_t last_bucket;
  {
    const uint32_t hi = ((uint32_t)(s_w[kLast] + 1) << drop) - 1u;
    const uint32_t lim = min((hi >> ib) + (uint32_t)E, 0xFFFFFFFFu >> ib);
    last_bucket = ((lim << ib) | mask) >> drop;
    int kept = 0;
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      if (u * NTHR >= have) continue;                       // uniform
      const bool keep = ((on >> u) & 1u) && (w[u] >> drop) <= last_bucket;
      uint32_t b = 0;
      if (keep) {
        b = bucket[w[u] >> drop];
        scat[(b & 0xFFFFu) + pos[u]] = w[u];
      } else {
        on &= ~(1u << u);
      }
      pos[u] = b;                                           // (from here on: start and size of the entry's bucket)
      kept += __popcll(__ballot(keep));
    }
    if (lane == 0) atomicAdd(&s_w[kKept], kept);
    if (__any((int)(last_bucket - s_w[kLast]) > 0)) {       // (buckets behind the kk-th's that are kept may be full as well)
      bool full = false;
#pragma unroll
      for (int u = 0; u < EPT; ++u) full = full || (((on >> u) & 1u) && (pos[u] >> 16) > (uint32_t)SIDE);
      if (full) s_w[kCrowded] = 1;
    }
  }
  __syncthreads();
  const int kept = s_w[kKept];
  if (s_w[kCrowded]) {
    // some bucket holds more than the rounds below sort (many near-equal values): count mates instead
#pragma unroll
    for (int u = 0; u < EPT; ++u)
      if ((on >> u) & 1u) {
        const int beg = (int)(pos[u] & 0xFFFFu), end = beg + (int)(pos[u] >> 16);
        int at = beg;
        for (int m = beg; m < end; ++m) at += scat[m] < w[u] ? 1 : 0;
        sorted[at] = w[u];
      }
    __syncthreads();
    for (int p = tid; p < kept; p += NTHR) scat[p] = sorted[p];
    __syncthreads();
  }
  constexpr int WIN = 128 - 2 * SIDE;
  for (int base = wv * WIN; base < kept; base += NTHR / 64 * WIN) {
    const int p = base - SIDE + 2 * lane;                   // my two entries (reads before and behind the entries stay inside the buffers)
    uint32_t x0 = scat[p], x1 = scat[p + 1];
    x0 = p < 0 ? 0u : (p >= kept ? 0xFFFFFFFFu : x0);
    x1 = p < 0 ? 0u : (p + 1 >= kept ? 0xFFFFFFFFu : x1);
#pragma unroll
    for (int r = 0; r < SIDE / 2; ++r) {
      const uint32_t lo = min(x0, x1), hi = max(x0, x1);
      // my second with the next lane's first, my first with the previous lane's second
      x1 = min(hi, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)lo, 0x130, 0xf, 0xf, false));
      x0 = max(lo, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x138, 0xf, 0xf, false));
    }
    const uint32_t px = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x1, 0x138, 0xf, 0xf, false);
    const int prev = (int)(px >> ib);
    const int next = (int)((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x0, 0x130, 0xf, 0xf, false) >> ib);
    const int v0 = (int)(x0 >> ib), v1 = (int)(x1 >> ib);
    const bool mid = p + 1 < kept && v1 - v0 <= E;
    const bool near0 = (p > 0 && v0 - prev <= E) || mid, near1 = mid || (p + 2 < kept && next - v1 <= E);
    // (long rows) entries that are the same code as the one before them go to the other end of the list, in which the
    // others then stand close: a block's turns at them are full ones
    auto put = [&](int q, bool follows) {
      if (STAGED && follows) {
        todo[sh.P - 1 - atomicAdd(&s_w[kFollow], 1)] = (uint16_t)q;
        atomicOr(&s_same[q >> 5], 1u << (q & 31));
      } else {
        todo[atomicAdd(&s_w[kTodo], 1)] = (uint16_t)q;
      }
    };
    if (lane >= SIDE / 2 && lane < 64 - SIDE / 2 && p < kept) {
      bool follows0 = false, follows1 = false;
      if (STAGED) {
        const bool even0 = near0 && p > 0 && (px ^ x0) >> ib == 0, even1 = near1 && (x0 ^ x1) >> ib == 0;
        if (even0 || even1) {
          const int t0 = R.twin[~x0 & mask];
          follows0 = even0 && R.twin[~px & mask] == t0;
          follows1 = even1 && R.twin[~x1 & mask] == t0;
        }
      }
      sorted[p] = x0;
      if (near0) put(p, follows0);
      else if (p < kk) out[1 + p] = (int32_t)(~x0 & mask);
      if (p + 1 < kept) {
        sorted[p + 1] = x1;
        if (near1) put(p + 1, follows1);
        else if (p + 1 < kk) out[2 + p] = (int32_t)(~x1 & mask);
      }
    }
  }
  __syncthreads();
  // an outsider lies below the threshold, value 0, and may be off by as much as any entry (and by the
  // rounding of the threshold)
  if (!all && (int)(~sorted[kk - 1] >> ib) <= E + 2) return false;      // uniform
  const int m = s_w[kTodo], mf = STAGED ? s_w[kFollow] : 0;
  auto follower = [&](int f) { return (int)todo[sh.P - 1 - f] & 0x7FFF; };
  // the first of the entries up to p, and the one behind those from p on, that are the same code
  auto run_start = [&](int p) {
    uint32_t w = (uint32_t)p >> 5, first = ~s_same[w] & (0xFFFFFFFFu >> (31 - (p & 31)));       // (entry 0 is never set)
    while (!first) first = ~s_same[--w];
    return (int)(32 * w) + 31 - __builtin_clz(first);
  };
  auto run_end = [&](int p) {
    int w = (p + 1) >> 5;
    uint32_t next = w < NTHR * EPT / 32 ? ~s_same[w] & (0xFFFFFFFFu << ((p + 1) & 31)) : 1u;
    while (!next) next = ++w < NTHR * EPT / 32 ? ~s_same[w] : 1u;
    return 32 * w + __builtin_ctz(next);
  };
  const bool chain = R.D <= kChainFloats && m + mf > NTHR / 8;      // uniform
  if (STAGED) {
    // Long rows: 16 lanes an entry, four floats of its row each per step,
    // their sums added across the lanes.  Such a sum and the key, which adds the same exact products in index order, are
    // each off by at most D 2^-53 of the products' magnitudes: where two sums are further
    // apart than `apart` (key_margin), the keys have the same order.  The few entries with a
    // closer one get their key.  Bound by waiting for the rows, of which few are in L2: what counts is the waves
    // in flight.  (A lane an entry, its row's pieces through 10 KB of LDS and 64 registers, left four blocks to a compute
    // unit and two of a block's four waves at work; now six blocks: 8192 x 256, k = 1000: the build 316 -> 269 us, 5000 x 96,
    // k = 2500: the build 403 -> 268.  The four chains of four lanes going round them, exact at once: 146 us.)
    // A code that is the same as the one before it in the order has that one's key and takes no part here.  (Every code
    // four times, the build: 8192 x 256, k = 1000: 0.94 ms with the look for them in the loop below, a lane in 16 asking, 0.50
    // so; 64 times 1.17 and 0.69; 1024 x 256, k = 100, four times: 83 us and 58.)
    const int l16 = lane & 15;
    if (chain) {
      for (int f = tid; f < m; f += NTHR) {
        const int p = todo[f];
        key[p] = exact_key(eid, R, (int)(~sorted[p] & mask));
      }
    } else {
      for (int f = tid >> 4; f < m; f += NTHR / 16) {
        const int p = todo[f];
        const float* r = R.p + (int64_t)(~sorted[p] & mask) * R.pitch;
        f32x4 x[4];
#pragma unroll
        for (int st = 0; st < 4; ++st)
          if (64 * st < R.D) x[st] = 64 * st + 4 * l16 < R.pitch ? *reinterpret_cast<const f32x4*>(r + 64 * st + 4 * l16) : f32x4{0.f, 0.f, 0.f, 0.f};
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int st = 0; st < 4; ++st)
          if (64 * st < R.D) {                                // uniform
            // (the row's floats out of LDS each time: in registers they cost more, in waves, than the reads do)
            const double* e = eid + min(64 * st + 4 * l16, R.pitch - 4);
            const f64x2 e0 = *reinterpret_cast<const f64x2*>(e), e1 = *reinterpret_cast<const f64x2*>(e + 2);
            s0 = __builtin_fma(e0[0], (double)x[st][0], s0);
            s1 = __builtin_fma(e0[1], (double)x[st][1], s1);
            s0 = __builtin_fma(e1[0], (double)x[st][2], s0);
            s1 = __builtin_fma(e1[1], (double)x[st][3], s1);
          }
        s0 = add_over_16(s0 + s1);
        if (l16 == 0) key[p] = orderable(s0);
      }
    }
    if (mf > 0) {                                           // uniform
      __syncthreads();
      for (int f = tid; f < mf; f += NTHR) key[follower(f)] = key[run_start(follower(f))];
    }
  } else {
    for (int f = tid; f < m; f += NTHR) {
      const int p = todo[f];
      key[p] = exact_key(eid, R, (int)(~sorted[p] & mask));
    }
  }
  __syncthreads();
  // the keys decide between entries that differ by at most E; all others are in order
  const double apart = STAGED && !chain ? key_margin(reach, R.D) : -1.0;
  auto place = [&](int p, bool sums) {                      // false: closer to some other than its sum tells
    const uint32_t x = sorted[p];
    const uint64_t K = key[p], lo = orderable(key_value(K) - apart), hi = orderable(key_value(K) + apart);
    const uint32_t I = ~x & mask;
    const int v = (int)(x >> ib);
    // (the entries of one value lie by descending index: a run of the same code is turned round)
    const int beg = STAGED ? run_start(p) : p, end = STAGED ? run_end(p) : p + 1;
    bool clear = true;
    int at = beg + end - 1 - p;
    for (int s = beg - 1; s >= 0; --s) {
      const uint32_t y = sorted[s];
      if (v - (int)(y >> ib) > E) break;
      const uint64_t L = key[s];
      clear = clear && (L < lo || L > hi);
      at -= before(L, ~y & mask, K, I) ? 0 : 1;
    }
    for (int s = end; s < kept; ++s) {
      const uint32_t y = sorted[s];
      if ((int)(y >> ib) - v > E) break;
      const uint64_t L = key[s];
      clear = clear && (L < lo || L > hi);
      at += before(L, ~y & mask, K, I) ? 1 : 0;
    }
    clear = clear || !STAGED || !sums || apart < 0.0;
    if (clear && at < kk) out[1 + at] = (int32_t)I;
    return clear;
  };
  // (what a run's first entry is told holds for all of it)
  bool unclear = false;
  for (int f = tid; f < m + mf; f += NTHR) {
    uint16_t& t = todo[f < m ? f : sh.P - 1 - (f - m)];
    if (!place(t, true)) { t |= 0x8000; unclear = true; }
  }
  if (STAGED && __syncthreads_or(unclear)) {
    for (int f = tid; f < m; f += NTHR)
      if (todo[f] & 0x8000) {
        const int p = todo[f] & 0x7FFF;
        key[p] = exact_key(eid, R, (int)(~sorted[p] & mask));
      }
    __syncthreads();
    if (mf > 0) {
      for (int f = tid; f < mf; f += NTHR) key[follower(f)] = key[run_start(follower(f))];
      __syncthreads();
    }
    for (int f = tid; f < m + mf; f += NTHR) {
      const int t = todo[f < m ? f : sh.P - 1 - (f - m)];
      if (t & 0x8000) place(t & 0x7FFF, false);
    }
  }
  return true;
}

// Rank of each of the n entries of (skey, sidx) in the order (key desc, idx asc), without a
// comparison sort: the keys are spread over NB buckets by a monotone map of their value
// (bucket 0 = largest), bucket sizes are scanned, the entries' ids are scattered bucket by
// bucket, and an entry's rank is its bucket's start plus the number of bucket mates that go
// before it.  The first kk ranks are written to out[1 + rank].  cur[NB] and ord[n] are LDS
// scratch, NB a multiple of NTHR.  Part of the exact path.
template <int NTHR>
__device__ void bucket_rank(const uint64_t* skey, const uint16_t* sidx, int n, int NB, uint32_t* cur, uint16_t* ord,
                            uint64_t* s_red, int* s_w, int kk, int32_t* out, int tid) {
  const int lane = tid & 63, wv = tid >> 6;
  uint64_t lo = ~0ull, hi = 0ull;
  for (int c = tid; c < n; c += NTHR) {
    const uint64_t K = skey[c];
    lo = K < lo ? K : lo;
    hi = K > hi ? K : hi;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t l2 = __shfl_xor(lo, o), h2 = __shfl_xor(hi, o);
    lo = l2 < lo ? l2 : lo;
    hi = h2 > hi ? h2 : hi;
  }
  if (lane == 0) { s_red[2 * wv] = lo; s_red[2 * wv + 1] = hi; }
  for (int b = tid; b < NB; b += NTHR) cur[b] = 0u;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NTHR / 64; ++w) {
    lo = s_red[2 * w] < lo ? s_red[2 * w] : lo;
    hi = s_red[2 * w + 1] > hi ? s_red[2 * w + 1] : hi;
  }
  const double xlo = key_value(lo), xhi = key_value(hi);
  const double span = xhi - xlo;
  // span may be 0, inf or NaN (equal, infinite or NaN keys): then everything shares bucket 0
  const double scale = (span > 0.0 && span < 1.0e300) ? (double)NB / span : 0.0;
  auto bucket_of = [&](uint64_t K) -> int {
    const double f = (xhi - key_value(K)) * scale;        // monotone non-increasing in K
    int b = f >= (double)(NB - 1) ? NB - 1 : (int)f;
    return f > 0.0 ? b : 0;                                // NaN and negatives to bucket 0
  };
  for (int c = tid; c < n; c += NTHR) atomicAdd(&cur[bucket_of(skey[c])], 1u);
  __syncthreads();
  {
    const int per = NB / NTHR;
    uint32_t local = 0u;
    for (int j = 0; j < per; ++j) local += cur[tid * per + j];
    int total;
    uint32_t run = (uint32_t)block_exclusive<NTHR>((int)local, s_w, tid, total);
    for (int j = 0; j < per; ++j) {
      const uint32_t cnt = cur[tid * per + j];
      cur[tid * per + j] = run;
      run += cnt;
    }
  }
  __syncthreads();
  for (int c = tid; c < n; c += NTHR) {
    const uint32_t pos = atomicAdd(&cur[bucket_of(skey[c])], 1u);
    ord[pos] = (uint16_t)c;
  }
  __syncthreads();
  // cur[b] is now the end of bucket b; its start is the end of bucket b - 1
  for (int c = tid; c < n; c += NTHR) {
    const uint64_t K = skey[c];
    const uint32_t I = sidx[c];
    const int b = bucket_of(K);
    const int beg = b ? (int)cur[b - 1] : 0, end = (int)cur[b];
    int rank = beg;
    for (int m = beg; m < end; ++m) {
      const int o = ord[m];
      rank += before(skey[o], sidx[o], K, I) ? 1 : 0;
    }
    if (rank < kk) out[1 + rank] = (int32_t)I;
  }
}

// LDS of the exact path in a block of `threads`, in bytes; keys: those of all codes are kept there.
size_t exact_lds(int V, int PD, int kk, int threads, bool keys) {
  return (size_t)PD * 8 + lpp_align_up((size_t)kk, threads) * 16 + 2 * 16 * 8 + 260 * 4 + (keys ? (size_t)V * 8 : 0);
}

// Exact path of one row over all V codes: radix select of the kk-th largest key.  KEEP: the keys are formed once
// and kept in LDS, not formed again in each of nine passes.  U: how many a thread forms side by side (rows of
// more than 16 floats: two; one takes fewer registers).
template <int NTHR, bool KEEP, int U>
__device__ void exact_row(const Rows& R, int V, int i, int kk, unsigned char* smem, int* s_w, int32_t* out, int tid) {
  const int lane = tid & 63, wv = tid >> 6;
  const int P = (kk + NTHR - 1) / NTHR * NTHR;
  double* eid = reinterpret_cast<double*>(smem);            // (already there)
  uint64_t* skey = reinterpret_cast<uint64_t*>(eid + ((R.D + 3) & ~3));
  uint32_t* cur = reinterpret_cast<uint32_t*>(skey + P);
  uint16_t* sidx = reinterpret_cast<uint16_t*>(cur + P);
  uint16_t* ord = sidx + P;
  uint64_t* s_red = reinterpret_cast<uint64_t*>(ord + P);   // [2 NTHR / 64]
  int* s_hist = reinterpret_cast<int*>(s_red + 2 * 16);
  int* s_misc = s_hist + 256;
  uint64_t* kept = reinterpret_cast<uint64_t*>(s_misc + 4);
  // keys of the codes j0 + u NTHR + tid (of the last one again past the end)
  auto form = [&](int j0, uint64_t (&K)[U]) {
    int j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) j[u] = min(j0 + u * NTHR + tid, V - 1);
    if (U == 1) K[0] = exact_key(eid, R, j[0]);
    else exact_keys<U>(eid, R, j, K);
  };
  if (KEEP)                                                 // (every thread reads back what it wrote itself)
    for (int j0 = 0; j0 < V; j0 += U * NTHR) {
      uint64_t K[U];
      form(j0, K);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (j0 + u * NTHR + tid < V) kept[j0 + u * NTHR + tid] = K[u];
    }
  auto keys = [&](int j0, uint64_t (&K)[U]) {
    if (!KEEP) form(j0, K);
#pragma unroll
    for (int u = 0; KEEP && u < U; ++u) K[u] = kept[min(j0 + u * NTHR + tid, V - 1)];
  };
  uint64_t prefix = 0ull;
  int need = kk;
  for (int byte = 7; byte >= 0; --byte) {
    __syncthreads();
    for (int t = tid; t < 256; t += NTHR) s_hist[t] = 0;
    __syncthreads();
    for (int j0 = 0; j0 < V; j0 += U * NTHR) {
      uint64_t K[U];
      keys(j0, K);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u * NTHR + tid;
        const bool match = j < V && j != i && (byte == 7 || (K[u] >> (8 * (byte + 1))) == (prefix >> (8 * (byte + 1))));
        const int digit = (int)((K[u] >> (8 * byte)) & 255ull);
        // (the bytes of keys that brought a row here are mostly the same: those of the wave's first in one add)
        const unsigned long long in = __ballot(match);
        if (in) {
          const int first = __builtin_ctzll(in), d0 = __builtin_amdgcn_readlane(digit, first);
          const unsigned long long same = __ballot(match && digit == d0);
          if (lane == first) atomicAdd(&s_hist[d0], __popcll(same));
          else if (match && digit != d0) atomicAdd(&s_hist[digit], 1);
        }
      }
    }
    __syncthreads();
    if (wv == 0) {                                          // lane: four bins, from the top
      int c[4], local = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) { c[b] = s_hist[255 - 4 * lane - b]; local += c[b]; }
      int above = local;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(above, o);
        if (lane >= o) above += t;
      }
      above -= local;
      if (above < need && above + local >= need) {
        int b = 0;
        for (; b < 3 && above + c[b] < need; ++b) above += c[b];
        s_misc[0] = 255 - 4 * lane - b;
        s_misc[1] = need - above;
      }
    }
    __syncthreads();
    prefix |= (uint64_t)s_misc[0] << (8 * byte);
    need = s_misc[1];
  }
  // prefix = exact kk-th largest key; keep everything above it plus the `need`
  // lowest-index codes equal to it
  const int n_gt = kk - need;
  __syncthreads();
  if (tid == 0) { s_misc[2] = 0; s_misc[3] = 0; }
  __syncthreads();
  for (int j0 = 0; j0 < V; j0 += U * NTHR) {
    uint64_t K[U];
    keys(j0, K);
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * NTHR + tid;
      const uint64_t key = U == 2 && u == 1 ? K[U - 1] : K[0];
      const bool other = j < V && j != i, gt = other && key > prefix, eq = other && key == prefix;
      if (gt) {
        const int pos = atomicAdd(&s_misc[2], 1);
        skey[pos] = key; sidx[pos] = (uint16_t)j;
      }
      // ordered compaction of the ties (ascending index)
      const unsigned long long bal = __ballot(eq);
      if (lane == 0) s_hist[wv] = __popcll(bal);
      __syncthreads();
      int base = s_misc[3];
      for (int w = 0; w < wv; ++w) base += s_hist[w];
      const int rank = base + __popcll(bal & ((1ull << lane) - 1ull));
      if (eq && rank < need) { skey[n_gt + rank] = key; sidx[n_gt + rank] = (uint16_t)j; }
      __syncthreads();
      if (tid == 0) {
        int t = 0;
        for (int w = 0; w < NTHR / 64; ++w) t += s_hist[w];
        s_misc[3] += t;
      }
      __syncthreads();
    }
  }
  bucket_rank<NTHR>(skey, sidx, kk, P, cur, ord, s_red, s_w, kk, out, tid);
}

// One block per row: NTHR threads, EPT list words each in registers.  A row that its list does not decide takes the
// exact path here, or (LATER) in a launch of its own.
// (Waves a SIMD asked for: what the LDS leaves room for; with the exact path of long rows inside, 64 registers are not
// enough, and scratch memory would cost every launch 1 us: blocks of 16 waves gain more by running in pairs, 5000 x 96,
// k = 2500: 314 -> 230 us.)
template <int NTHR, int EPT, bool STAGED, bool LATER>
__global__ __launch_bounds__(NTHR, LATER || !STAGED || NTHR == 1024 ? 8 : 6) void knn_rank_kernel(KnnArgs a, RankShape sh) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_w[STAGED ? 24 : 20];
  const int tid = threadIdx.x, i = blockIdx.x, kk = a.k - 1;
  int32_t* out = a.neigh + (int64_t)i * a.k;
  if (tid == 0) out[0] = i;
  if (kk == 0) return;
  const RowPlan p = a.plan[i];
  const uint32_t* list = a.cand + (int64_t)i * a.cap;
  const uint32_t mask = (1u << a.ib) - 1u;
  uint32_t w[EPT], on = 0;
  const int n = a.cnt[i];
  const bool over = n > a.cap;                              // uniform: the list does not hold everything it should
#pragma unroll
  for (int u = 0; u < EPT; ++u) w[u] = 0;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int c = tid + u * NTHR;
    if (u * NTHR < n && c < min(n, a.cap)) w[u] = list[c];
  }
  double* eid = reinterpret_cast<double*>(smem);
  for (int d = tid; d < a.PD; d += NTHR) eid[d] = (double)a.Ep[(int64_t)i * a.PD + d];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    if (u * NTHR >= n) continue;                            // uniform
    const uint32_t j = w[u] & mask;                         // the row itself and padding are no neighbours
    bool keep = tid + u * NTHR < n && j != (uint32_t)i && j < (uint32_t)a.V;
    if (keep && (p.flags & kAnyNan)) keep = a.norms[j] == a.norms[j];      // (a code that holds a NaN is no neighbour)
    on |= keep ? 1u << u : 0u;
    w[u] = ~w[u];
  }
  if (p.flags & kFlat) {                                    // uniform (here: the loads above do not wait for the plan)
    for (int t = tid; t < kk; t += NTHR) out[1 + t] = t < i ? t : t + 1;
    return;
  }
  const Rows R{a.Ep, a.PD, a.D, true, a.twin};
  if (!over && !(p.flags & kNoList)) {
    if (rank_row<NTHR, EPT, STAGED>(w, on, n, a.ib, a.vmask_bits, p.E, (p.flags & kAll) != 0, kk, R,
                                   STAGED ? a.reach[i] : 0.f, sh, smem, s_w, out, tid)) return;
  }
  // (what was written of the row is written again)
  if constexpr (LATER) {
    if (tid == 0) a.redo[1 + atomicAdd(a.redo, 1)] = i;
  } else {
    __threadfence();
    __syncthreads();
    exact_row<NTHR, false, STAGED ? 2 : 1>(R, a.V, i, kk, smem, s_w, out, tid);
  }
}

// The rows that no list decides, one after the other by blocks of 16 waves: 0.02 to 0.1 ms a row (D = 8), 0.3 ms
// (D = 256); inside the ranking's blocks it is 0.4 to 0.9 ms and 2 to 9 ms.
constexpr int kExactThreads = 1024;
template <bool KEEP>
__global__ __launch_bounds__(kExactThreads) void knn_exact_kernel(KnnArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_w[20];
  const int n = a.redo[0];
  for (int r = blockIdx.x; r < n; r += gridDim.x) {
    const int i = a.redo[1 + r];
    double* eid = reinterpret_cast<double*>(smem);
    for (int d = threadIdx.x; d < a.PD; d += kExactThreads) eid[d] = (double)a.Ep[(int64_t)i * a.PD + d];
    __syncthreads();
    exact_row<kExactThreads, KEEP, KEEP ? 2 : 1>(Rows{a.Ep, a.PD, a.D, true, a.twin}, a.V, i, a.k - 1, smem, s_w, a.neigh + (int64_t)i * a.k, threadIdx.x);
    __syncthreads();
  }
}

// Small codebooks of short rows: one block per row forms the row's similarities with every code
// (fp32, in registers) and ranks them; nothing goes through memory but the codebook and the row.
constexpr int kDirectThreads = 256;
__global__ __launch_bounds__(kDirectThreads) void knn_direct_kernel(KnnArgs a, RankShape sh) {
  constexpr int EPT = kDirectCodes / kDirectThreads, W = kDirectThreads / 64;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_w[20];
  __shared__ float s_m[3][W];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, i = blockIdx.x, kk = a.k - 1;
  const int D = a.D, V = a.V;
  int32_t* out = a.neigh + (int64_t)i * a.k;
  if (tid == 0) out[0] = i;
  if (kk == 0) return;
  double* eid = reinterpret_cast<double*>(smem);
  const int PD = (D + 3) & ~3;
  if (tid < PD) eid[tid] = tid < D ? (double)a.E[(int64_t)i * D + tid] : 0.0;
  const bool quads = (D & 3) == 0 && (reinterpret_cast<uintptr_t>(a.E) & 15) == 0;
  float q[kShortRow];                                       // (uniform: scalar loads)
#pragma unroll
  for (int d = 0; d < kShortRow; ++d) q[d] = d < D ? a.E[(int64_t)i * D + d] : 0.f;
  float sim[EPT], lo = INFINITY, hi = -INFINITY, maxn2 = 0.f;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int c = min(tid + u * kDirectThreads, V - 1);
    const float* e = a.E + (int64_t)c * D;
    float s = 0.f, n2 = 0.f;
    if (quads) {
#pragma unroll
      for (int t = 0; t < kShortRow; t += 4)
        if (t < D) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(e + t);
#pragma unroll
          for (int x = 0; x < 4; ++x) { s = __builtin_fmaf(q[t + x], v[x], s); n2 = __builtin_fmaf(v[x], v[x], n2); }
        }
    } else {
#pragma unroll
      for (int t = 0; t < kShortRow; ++t)
        if (t < D) { const float v = e[t]; s = __builtin_fmaf(q[t], v, s); n2 = __builtin_fmaf(v, v, n2); }
    }
    sim[u] = s;
    maxn2 = fmaxf(maxn2, n2);
    lo = fminf(lo, s);
    hi = fmaxf(hi, s);
  }
  lo = -lo;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmaxf(lo, __shfl_xor(lo, o));
    hi = fmaxf(hi, __shfl_xor(hi, o));
    maxn2 = fmaxf(maxn2, __shfl_xor(maxn2, o));
  }
  if (lane == 0) { s_m[0][wv] = lo; s_m[1][wv] = hi; s_m[2][wv] = maxn2; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < W; ++w) { lo = fmaxf(lo, s_m[0][w]); hi = fmaxf(hi, s_m[1][w]); maxn2 = fmaxf(maxn2, s_m[2][w]); }
  lo = -lo;
  if (__builtin_expect(hi == 0.f && lo == 0.f, 0)) {        // uniform
    // a row of zeros, no similarity a NaN: the lowest codes (1024 x 8, 30 % zeros: 1072 -> 9 us)
    bool other = false;
#pragma unroll
    for (int u = 0; u < EPT; ++u) other = other || sim[u] != 0.f;
#pragma unroll 1
    for (int d = 0; d < D; ++d) other = other || eid[d] != 0.0;
    if (!__syncthreads_or(other)) {
      for (int t = tid; t < kk; t += kDirectThreads) out[1 + t] = t < i ? t : t + 1;
      return;
    }
  }
  float n2 = 0.f;
#pragma unroll
  for (int d = 0; d < kShortRow; ++d) n2 = __builtin_fmaf(q[d], q[d], n2);
  const float qmax = (float)((1u << a.vmask_bits) - 2u);
  // (the float product of the norms may underflow where the keys do not: a floor keeps E on the safe side)
  const float e = (float)(PD + 4) * 1.1920929e-07f * sqrtf(n2) * sqrtf(maxn2) * 1.001f + 1e-36f;
  const float range = fmaxf(hi - lo, fmaxf(e, 1e-30f));
  const float pa = qmax / range, pb = 1.0f - lo * pa;
  const int E = (int)fminf(ceilf(2.002f * e * pa) + 4.0f, 1073741824.0f);
  uint32_t w[EPT], on = 0;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int c = tid + u * kDirectThreads;
    w[u] = ~(((uint32_t)fminf(fmaxf(__builtin_fmaf(sim[u], pa, pb), 0.f), qmax) << a.ib) | (uint32_t)c);
    on |= c < V && c != i && sim[u] == sim[u] ? 1u << u : 0u;      // (a code that holds a NaN is no neighbour)
  }
  __syncthreads();
  const Rows R{a.E, D, D, quads, nullptr};
  if (range < INFINITY && rank_row<kDirectThreads, EPT, false>(w, on, V, a.ib, a.vmask_bits, E, true, kk, R, 0.f, sh, smem, s_w, out, tid))
    return;
  __threadfence();                                          // (what was written of the row is written again by other lanes)
  __syncthreads();
  exact_row<kDirectThreads, false, 1>(R, V, i, kk, smem, s_w, out, tid);
}

// -------------------------------------------------------------------------------------------- host

struct KnnLayout {
  size_t o_ep, o_ef, o_es, o_ew, o_ews, o_norms, o_l1, o_hash, o_seen, o_twin, o_part, o_plan, o_reach, o_cnt, o_redo, o_cand, total;
  int32_t PD, KS, Vp, cap, ib, vb, stride, ns, m, take_all, most, splits, seen_shift;
};

int log2_up(int x) { int l = 0; while ((1 << l) < x) ++l; return l; }

KnnLayout knn_layout(int32_t V, int32_t D, int32_t k) {
  KnnLayout L;
  L.PD = (D + 3) & ~3;
  L.KS = D > kShortRow ? (D + 63) / 64 : 0;
  L.Vp = (int32_t)lpp_align_up((size_t)V, 128);
  L.ib = 8;
  while ((1 << L.ib) < L.Vp && L.ib < 16) ++L.ib;
  L.vb = 32 - L.ib;
  // The sample: codes above the k - 1 th largest are in it with probability 1 / stride each; the
  // m-th largest of the sample lies below that one unless the sample holds five standard deviations
  // too many of them (the z^2 / 4 term is for counts so small that they are not normal; 1.05 leaves
  // some spread where the sample is the whole codebook: its similarities are rounded).
  const int kk = k - 1;
  L.stride = 1;
  while (L.stride * 2 * kSampleCodes <= V) L.stride *= 2;
  L.ns = V / L.stride;
  const double mu = (double)kk / L.stride, z = 5.0;
  L.m = (int)ceil(mu + z * sqrt(mu * (1.05 - 1.0 / L.stride)) + z * z / 4.0) + 1;
  const double expect = (double)L.m * L.stride, dev = L.stride * sqrt((double)L.m * (1.0 - 0.999 / L.stride));
  L.take_all = expect >= 0.75 * V;
  // (the last term: the threshold is the lower edge of a bin, whose codes are all taken)
  L.cap = L.take_all ? L.Vp : (int32_t)std::min<size_t>(L.Vp, lpp_align_up((size_t)(expect + 5.0 * dev) + 64 + V / 256, 64));
  L.most = L.m + (int)std::max(0.0, (L.cap - expect) / (2.0 * L.stride));
  // long rows: blocks of 128 queries by `splits` shares of the code tiles, two blocks per compute unit
  const int groups = L.Vp / 128;
  L.splits = L.KS ? std::max(1, std::min({2 * kUnits / groups, 8 * (groups / 2 + 1), kMaxSplits})) : 1;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o += lpp_align_up(bytes, 256); return at; };
  L.o_ep = take((size_t)V * L.PD * sizeof(float));
  const int n8 = D > 8 ? 2 : 1;
  L.o_ef = take(L.KS ? (size_t)(L.Vp / 16) * L.KS * 3 * 64 * 16 : (size_t)L.Vp * 2 * n8 * 16);
  L.o_es = take(L.KS ? (size_t)((L.ns + 15) / 16) * L.KS * 64 * 16 : lpp_align_up((size_t)L.ns, 16) * 2 * n8 * 16);
  L.o_ew = take(L.KS ? 0 : (size_t)L.Vp * 2 * n8 * 16);
  L.o_ews = take(L.KS ? 0 : lpp_align_up((size_t)L.ns, 16) * 2 * n8 * 16);
  L.o_norms = take((size_t)V * sizeof(float));
  L.o_l1 = take((size_t)V * sizeof(float));
  L.o_hash = take(L.KS ? (size_t)V * sizeof(uint32_t) : 0);
  L.seen_shift = 32 - log2_up(std::max(V, 1024)) - 2;
  L.o_seen = take(L.KS ? sizeof(int32_t) << (33 - L.seen_shift) : 0);
  L.o_twin = take(L.KS ? (size_t)V * sizeof(int32_t) : 0);
  L.o_part = take((size_t)kStatBlocks * sizeof(float4));
  L.o_plan = take((size_t)L.Vp * sizeof(RowPlan));
  L.o_reach = take(L.KS ? (size_t)L.Vp * sizeof(float) : 0);
  L.o_cnt = take((size_t)V * sizeof(int32_t));
  L.o_redo = take((size_t)(V + 1) * sizeof(int32_t));
  L.o_cand = take((size_t)V * L.cap * sizeof(uint32_t));
  L.total = o;
  return L;
}

// LDS of one row's ranking
size_t rank_lds(int P, int NB, int PD) { return (size_t)PD * 8 + (size_t)NB * 4 + (size_t)P * 8 + (size_t)P * 2; }

template <bool FIXED, int N, int NQ>
int32_t launch_sample_as(const KnnArgs& a, hipStream_t s) {
  const size_t lds = (size_t)kSampleBins * 16 * sizeof(uint32_t);
  auto kern = knn_sample_kernel<FIXED, N, NQ>;
  static LppLdsLimit limit;
  const int32_t st = lpp_ensure_lds(reinterpret_cast<const void*>(kern), limit, lds);
  if (st != LPP_OK) return st;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.Vp / (16 * NQ))), dim3(kSampleThreads), lds, s, a);
  LPP_HIP_TRY(hipGetLastError());
  return LPP_OK;
}
// 32 rows a block where blocks of 16 would come in more turns than one; both sides, the build: 16384 x 16, k = 1000 247.5 us
// (16 rows) and 232.0 (32), 12000 x 13, k = 300 136.9 and 129.3, but 8192 x 8, k = 16 46.7 and 48.0, 4096 x 8, k = 100 29.9
// and 34.3.  Rows of more than 64 floats already where some compute unit gets a second block (two of 16 rows are there at once,
// but each reads all of the sample): 6001 x 129, k = 300 109.2 and 103.9, 8192 x 256, k = 1000 196.3 and 188.9; up to 64
// floats it gives nothing: 8192 x 64, k = 100 81.5 and 82.7, 12000 x 64 151.9 and 153.2, 16384 x 64, k = 1000 329.9 and 328.6.
template <bool FIXED, int N>
int32_t launch_sample(const KnnArgs& a, hipStream_t s) {
  if constexpr (!FIXED || N > 1)
    if (a.Vp > (FIXED ? 16 : 32) * kUnits) return launch_sample_as<FIXED, N, 2>(a, s);
  return launch_sample_as<FIXED, N, 1>(a, s);
}

template <int N>
int32_t launch_collect_f16(const KnnArgs& a, hipStream_t s) {
  int32_t st = launch_sample<false, N>(a, s);
  if (st != LPP_OK) return st;
  // a block per 16 queries: as many waves as give every compute unit 18 (8 KB of LDS each), 16 at most
  const int blocks = (a.V + 15) / 16;
  const int waves = std::max(4, std::min(kCollectMaxWaves, kUnits * 18 / blocks));
  const size_t lds = (size_t)waves * 8192;
  auto kern = knn_collect_f16_kernel<N>;
  static LppLdsLimit limit;
  st = lpp_ensure_lds(reinterpret_cast<const void*>(kern), limit, lds, 48 * 1024);
  if (st != LPP_OK) return st;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3((unsigned)waves * 64), lds, s, a);
  LPP_HIP_TRY(hipGetLastError());
  return LPP_OK;
}

template <int KS>
int32_t launch_collect_i8(const KnnArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(knn_limb_kernel<KS>, dim3((unsigned)(a.Vp / 16 * KS / 4)), dim3(256), 0, s, a);
  LPP_HIP_TRY(hipGetLastError());
  int32_t st = launch_sample<true, KS>(a, s);
  if (st != LPP_OK) return st;
  hipLaunchKernelGGL(knn_collect_i8_kernel<KS>, dim3((unsigned)(a.Vp / (kCollectWaves * 32) * a.splits)),
                     dim3(kCollectWaves * 64), 0, s, a);
  LPP_HIP_TRY(hipGetLastError());
  return LPP_OK;
}

// Every key of a row in LDS where they fit (16384 codes and k = 1000, or 8192 and 4096).
template <bool KEEP>
int32_t launch_exact_as(const KnnArgs& a, hipStream_t s) {
  const size_t lds = exact_lds(a.V, a.PD, a.k - 1, kExactThreads, KEEP);
  auto kern = knn_exact_kernel<KEEP>;
  static LppLdsLimit limit;
  const int32_t st = lpp_ensure_lds(reinterpret_cast<const void*>(kern), limit, lds, 48 * 1024);
  if (st != LPP_OK) return st;
  hipLaunchKernelGGL(kern, dim3((unsigned)std::min(a.V, kUnits)), dim3(kExactThreads), lds, s, a);
  LPP_HIP_TRY(hipGetLastError());
  return LPP_OK;
}
int32_t launch_exact(const KnnArgs& a, hipStream_t s) {
  return exact_lds(a.V, a.PD, a.k - 1, kExactThreads, true) <= kMostLds ? launch_exact_as<true>(a, s) : launch_exact_as<false>(a, s);
}

template <int NTHR, bool STAGED, bool LATER>
int32_t launch_rank(const KnnArgs& a, RankShape sh, hipStream_t s) {
  const size_t own = rank_lds(sh.P, 1 << sh.lognb, a.PD);
  const size_t lds = LATER ? own : std::max(own, exact_lds(a.V, a.PD, a.k - 1, NTHR, false));
  if (lds > kMostLds) return LPP_EUNSUPPORTED;
  auto kern = knn_rank_kernel<NTHR, 8, STAGED, LATER>;
  static LppLdsLimit limit;
  const int32_t st = lpp_ensure_lds(reinterpret_cast<const void*>(kern), limit, lds, 48 * 1024);
  if (st != LPP_OK) return st;
  hipLaunchKernelGGL(kern, dim3((unsigned)a.V), dim3(NTHR), lds, s, a, sh);
  LPP_HIP_TRY(hipGetLastError());
  return LATER && a.k > 1 ? launch_exact(a, s) : LPP_OK;
}

}  // namespace

extern "C" size_t lpp_build_neighbours_workspace(int32_t V, int32_t D, int32_t k) {
  if (V < 1 || D < 1 || k < 1 || k > V || k > LPP_MAX_K || D > 256 || V > 65536) return 0;
  return knn_layout(V, D, k).total;
}

extern "C" int32_t lpp_build_neighbours(const float* E, int32_t V, int32_t D, int32_t k, int32_t* neigh,
                                        void* ws, size_t ws_bytes, void* stream) {
  if (!E || !neigh) return LPP_EINVAL;
  if (V < 1 || D < 1 || k < 1 || k > V) return LPP_EINVAL;
  if (k > LPP_MAX_K || D > 256 || V > 65536) return LPP_EUNSUPPORTED;
  const KnnLayout L = knn_layout(V, D, k);
  if (!ws || ws_bytes < L.total) return LPP_ENOWORKSPACE;
  static std::atomic<bool> have_device{false};
  if (!have_device.load(std::memory_order_relaxed)) {
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) { (void)hipGetLastError(); return LPP_EHIP; }
    have_device.store(true, std::memory_order_relaxed);
  }
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  unsigned char* w = reinterpret_cast<unsigned char*>(ws);
  KnnArgs a;
  a.E = E; a.V = V; a.D = D; a.k = k; a.PD = L.PD; a.Vp = L.Vp; a.cap = L.cap; a.ib = L.ib; a.vmask_bits = L.vb;
  a.stride = L.stride; a.ns = L.ns; a.m = L.m; a.take_all = L.take_all; a.most = L.most; a.splits = L.splits;
  const bool as_is = (D & 3) == 0 && (reinterpret_cast<uintptr_t>(E) & 15) == 0;
  a.copy = as_is ? nullptr : reinterpret_cast<float*>(w + L.o_ep);
  a.Ep = as_is ? E : a.copy;
  a.Ef = reinterpret_cast<i32x4*>(w + L.o_ef);
  a.Es = reinterpret_cast<i32x4*>(w + L.o_es);
  a.Ew = reinterpret_cast<i32x4*>(w + L.o_ew);
  a.Ews = reinterpret_cast<i32x4*>(w + L.o_ews);
  a.norms = reinterpret_cast<float*>(w + L.o_norms);
  a.l1 = reinterpret_cast<float*>(w + L.o_l1);
  a.hash = reinterpret_cast<uint32_t*>(w + L.o_hash);
  a.seen = reinterpret_cast<int32_t*>(w + L.o_seen);
  a.twin = reinterpret_cast<int32_t*>(w + L.o_twin);
  a.seen_shift = L.seen_shift;
  a.part = reinterpret_cast<float4*>(w + L.o_part);
  a.plan = reinterpret_cast<RowPlan*>(w + L.o_plan);
  a.reach = reinterpret_cast<float*>(w + L.o_reach);
  a.cnt = reinterpret_cast<int32_t*>(w + L.o_cnt);
  a.cand = reinterpret_cast<uint32_t*>(w + L.o_cand);
  a.redo = reinterpret_cast<int32_t*>(w + L.o_redo);
  a.neigh = neigh;

  if (D <= kShortRow && V <= kDirectCodes) {
    // values need no more than the float's bits; the key buffer over counters and scattered words wants NB >= P
    const RankShape sh{kDirectCodes, log2_up(kDirectCodes)};
    const size_t lds = std::max(rank_lds(sh.P, 1 << sh.lognb, L.PD), exact_lds(V, L.PD, k - 1, kDirectThreads, false));
    hipLaunchKernelGGL(knn_direct_kernel, dim3((unsigned)V), dim3(kDirectThreads), lds, s, a, sh);
    LPP_HIP_TRY(hipGetLastError());
    return LPP_OK;
  }

  const int G = D <= 16 ? 4 : (D <= 64 ? 16 : 64);
  a.statblocks = std::min(kStatBlocks, (V + kStatThreads / G - 1) / (kStatThreads / G));
  if (G == 4) hipLaunchKernelGGL(knn_stats_kernel<4>, dim3((unsigned)a.statblocks), dim3(kStatThreads), 0, s, a);
  else if (G == 16) hipLaunchKernelGGL(knn_stats_kernel<16>, dim3((unsigned)a.statblocks), dim3(kStatThreads), 0, s, a);
  else hipLaunchKernelGGL(knn_stats_kernel<64>, dim3((unsigned)a.statblocks), dim3(kStatThreads), 0, s, a);
  LPP_HIP_TRY(hipGetLastError());
  if (k > 1) {
    int32_t st;
    if (D <= kShortRow) {
      st = D <= 8 ? launch_collect_f16<1>(a, s) : launch_collect_f16<2>(a, s);
    } else {
      switch (L.KS) {
        case 1: st = launch_collect_i8<1>(a, s); break;
        case 2: st = launch_collect_i8<2>(a, s); break;
        case 3: st = launch_collect_i8<3>(a, s); break;
        default: st = launch_collect_i8<4>(a, s); break;
      }
    }
    if (st != LPP_OK) return st;
  }
  // a list of up to eight words per thread, which is as few waves as hold it: one, two, four or sixteen.  What a thread does
  // beside its words, and the barriers, cost more than fewer rows at once: lists of 513 to 1024 by two waves instead of four,
  // 16384 x 8, k = 200 133.4 -> 120.7 us, 4096 x 64, k = 500 63.3 -> 58.8, 8192 x 256, k = 300 150.3 -> 146.3,
  // 16384 x 64, k = 400 268.8 -> 253.8; up to 2048 by eight instead of four 186 -> 211 (16384 x 8, k = 1000), by two
  // with sixteen words each 186 -> 216.
  const bool staged = D > kShortRow;
  // Rows that fall through (heavy ties, infinities, norms far apart) in a launch of their own, which costs 2 us
  // whether there are any or not: where one such row would cost many times that in a ranking block (codebooks of 2^20
  // numbers of long rows), and where one wave ranks a row of a large codebook, whose blocks then hold the LDS of a
  // list only.  900 equal codes among 8192 x 256, k = 16, 300, 1000: 13.9, 28.4, 15.8 ms -> 1.4, 1.9, 3.4; all else
  // equal, 8192 x 256: k = 16 195 -> 182 us, 100 223 -> 202, 300 266.5 -> 268.4, 1000 316.8 -> 318.4; 16384 x 8:
  // k = 16 116 -> 99, 100 131 -> 114 us.  2048 x 8, k = 16: 23.6 us without, 25.8 with.
  const bool later = staged ? (int64_t)V * D > kLaterFloats : L.cap <= 512 && V > kLaterCodes;
  auto rank = [&](auto threads, int least) {
    constexpr int NTHR = decltype(threads)::value;
    const RankShape sh{L.cap, std::max(least, log2_up(L.cap))};
    if (staged) return later ? launch_rank<NTHR, true, true>(a, sh, s) : launch_rank<NTHR, true, false>(a, sh, s);
    return later ? launch_rank<NTHR, false, true>(a, sh, s) : launch_rank<NTHR, false, false>(a, sh, s);
  };
  if (L.cap <= 512) return rank(std::integral_constant<int, 64>(), 8);
  if (L.cap <= 1024) return rank(std::integral_constant<int, 128>(), 9);
  if (L.cap <= 2048) return rank(std::integral_constant<int, 256>(), 10);
  if (L.cap > 8192) return LPP_EUNSUPPORTED;
  return rank(std::integral_constant<int, 1024>(), 12);
}
