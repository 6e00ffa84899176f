// Tree-masked decode attention of the flattened draft tree against the target
// model's KV cache (paper Sec. 2.1; App. A.2 "Tree drafting and decoding": every
// tree row sees the whole prefix plus its ancestors and itself, nothing else).
//
// bf16 path.  Keys are cut into groups of 32 (cache groups first, then tree
// groups).  A wave owns whole groups and all tree rows of its block's row range:
//   S^T[32 keys x rows] = K_group * Q^T       (MFMA 16x16x32 bf16, K straight from HBM
//                                              into the A operand, Q held in registers)
//   softmax down the key axis, which is mostly lane-local in this layout; the
//   reference maximum of a row only moves when a score exceeds it by 2^8, so the
//   accumulators are rarely rescaled
//   O^T[Dh x rows]    += V_group^T * P^T       (V rows go to a wave-private LDS tile as
//                                              they are and come back through the
//                                              transposing LDS read; P stays in registers;
//                                              a tile of ones in place of V^T gives the
//                                              row sums of the rounded P)
// The loads of a wave's next group are issued before it works on the current one.
// The ancestor mask is one 64-bit word per (row, 64 tree keys) and only touches
// tree groups.  Waves of a block merge their (max, sum, O) through LDS; when the
// key range of one (batch, head) is split over several blocks to fill the chip the
// partials go through the workspace and the block that finishes last adds them up
// in split order.
//
// fp32 path: the same two products on the float32 matrix cores, straight from the loads.
#include <math.h>
#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "lpp_internal.h"
#include "lpp_reciprocal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr float kMasked = -1.0e30f;  // finite stand-in for -inf
// log2 of the largest probability weight before a rescale.  (Lower, long sweeps take longer: at 2^1, 129 rows, 4096 keys, 384 heads
// 107 -> 121 us.)
constexpr float kLazy = 8.0f;

// Several layers of one step go out in one launch: unit / units_per_layer picks the layer,
// whose tensors are looked up in a table inside the kernel arguments (a wave-uniform index).
constexpr int kLayersPerLaunch = 16;
struct LayerPtrs {
  const void* q; const void* kc; const void* vc; const void* kt; const void* vt;
  void* out;                         // [B,H,M,Dh] float, or bf16 when out_bf16
};

struct AttnArgs {
  // (what every block needs to find its place lies together: one line of the scalar cache)
  uint32_t units_per_layer, rc_upl;  // units of a layer: first those of its key/value heads in eights, then those of the heads left
  uint32_t eights;                   // ... units of the former
  uint32_t left, rc_left;            // key/value heads left, 0 to 7
  uint32_t spin;                     // ... none, the last eight padded: how far its heads move from layer to layer
  uint32_t whole_eights;             // the launch's units (layer, head, row range) in eights, and those left
  uint32_t units_left, rc_units_left;
  int32_t nsplit; uint32_t rc_nsplit;   // blocks of a unit: `share` for each of its key ranges
  int32_t ranges; uint32_t rc_ranges;
  int32_t share_bits;                // log2(share)
  int32_t msplits; uint32_t rc_msplits; // row ranges of a head.  rc_d: for div_rc; n d < 2^32 as blocks < 2^31, B H^2 < 2^32, msplits <= 8
                                     // (16 where the blocks are few), the layers as layers_per_launch has them
  int32_t gq; uint32_t rc_gq;        // query heads per key/value head (H = Hkv * gq)
  int32_t H; uint32_t rc_H;
  int32_t KVBH, S, M, words;         // KVBH: batch * key/value heads
  int32_t out_bf16;                  // out holds bf16 instead of float
  const int32_t* seq_len;
  const uint64_t* anc;
  float scale_log2;                  // scale * log2(e)
  uint32_t ws_o_bytes, ws_ml_bytes;  // sizes of the two, each below 2^31
  int32_t rows_pad;                  // ceil(M / 16) * 16
  float* ws_o;                       // [layer][BH][nsplit][rows_pad][Dh]   unnormalised partial O
  float* ws_ml;                      // [layer][BH][nsplit][rows_pad][2]    (reference max in log2 units, sum)
  int32_t* counters;                 // [unit] zero between calls
  LayerPtrs layer[kLayersPerLaunch];
};

// x, as something the compiler does not know: what is formed from it is formed here, and takes no registers
// (which the loops over the keys have none to spare of) before.
__device__ __forceinline__ int formed_anew(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ uint4 ld16(const char* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ uint4 ld16(const uint16_t* p) {
  return *reinterpret_cast<const uint4*>(p);
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {   // round to nearest even (hardware convert)
  const bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// 16- and 8-byte accesses that are visible device-wide once they have completed (the cache policy
// of a device-scope atomic, on whole vectors): what the blocks of one head exchange their partial
// results with inside one launch.  `off` is a byte offset into the buffer behind `rsrc`.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr int kDeviceScope = 16;     // sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t device_buffer(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void store_dev(__amdgpu_buffer_rsrc_t r, uint32_t off, float4 v) {
  const u32x4 x = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
  __builtin_amdgcn_raw_buffer_store_b128(x, r, (int)off, 0, kDeviceScope);
}
__device__ __forceinline__ void store_dev(__amdgpu_buffer_rsrc_t r, uint32_t off, float2 v) {
  const u32x2 x = {__float_as_uint(v.x), __float_as_uint(v.y)};
  __builtin_amdgcn_raw_buffer_store_b64(x, r, (int)off, 0, kDeviceScope);
}
__device__ __forceinline__ float4 load_dev4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kDeviceScope);
  return make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
}
__device__ __forceinline__ float2 load_dev2(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, kDeviceScope);
  return make_float2(__uint_as_float(x.x), __uint_as_float(x.y));
}

// four consecutive output elements starting at element index e of the output tensor
__device__ __forceinline__ void store_out4(float* out, bool as_bf16, int64_t e, float4 v) {
  if (as_bf16)
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + e) = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
  else
    *reinterpret_cast<float4*>(out + e) = v;
}

// One key group in flight: K as the A operand of S^T = K Q^T, V as loaded (row-major chunks).
template <int DH>
struct Stage {
  bf16x8 ka[2][DH / 32];
  uint4 vr[DH / 16];     // chunk c = lane + 64 p of the group's 32 x (DH/8) 16-byte chunks
};

// NT = row tiles (of 16 tree rows) per wave, RW = waves along the rows, KW = waves along the keys:
// a block covers NT * RW * 16 tree rows; of the KW * share waves of a key range wave w takes its groups gbeg + w, + KW * share, ... for
// rows [rw NT 16, (rw + 1) NT 16).  The RW waves that share a key group load it independently; the
// second read is served by the compute unit's own cache.
template <int DH, int NT, int RW, int KW>
__global__ __launch_bounds__(RW * KW * 64, (RW * KW == 4 ? (NT <= 2 && DH == 64 ? (NT == 1 ? 4 : 3) : 2) : 1)) void tree_attn_bf16_kernel(AttnArgs a) {
  static_assert(RW == 1, "a block is one row range; its waves split the keys");
  constexpr int W = RW * KW;
  constexpr int KS = DH / 32;        // contraction steps of Q K^T
  constexpr int DT = DH / 16;        // Dh tiles of the output
  constexpr int CPR = DH / 8;        // 16-byte chunks per K/V row
  constexpr int VCH = DH / 16;       // V chunks per lane and group
  constexpr int VPITCH = DH * 2 + 32;   // bytes per key of the LDS V tile: 32 mod 256, so that the
                                        // 16 keys x 32 bytes of a transposing read hit all banks once
  constexpr int VTILE = 32 * VPITCH;
  constexpr int WROWS = NT * 16;     // rows of a wave
  constexpr int ROWS = RW * WROWS;   // rows of the block
  constexpr int OPITCH = DH + 4;     // floats per row of the merge buffer
  constexpr bool kLean = DH != 64 || NT >= 5;   // no registers for a third stage
  // merge slots: one per wave if that fits where the V tiles were (or in 12 KB per wave), else half as many
  constexpr int MS = (KW * NT * 16 * (DH + 4) * 4 <= (KW * 2 * VTILE > KW * 12 * 1024 ? KW * 2 * VTILE : KW * 12 * 1024)) ? KW : KW / 2;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_ticket;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int kw = wave % KW, rw = wave / KW;

  // block -> unit = (layer, batch*head, row range) and key range; all blocks of one key/value head (every row range
  // and every query head that reads it) share an XCD, as long as all XCDs have one, and follow each other in launch order
  // (Every argument is asked for at once, then the layer's pointers and the item's length, and no branch up to the first
  // loads: left to the compiler, the scalar loads wait for each other four times, a few tenths of a microsecond each.)
  uint32_t upl = a.units_per_layer, rc_upl = a.rc_upl, eights = a.eights, left = a.left, rc_left = a.rc_left, spin = a.spin;
  uint32_t whole_eights = a.whole_eights, units_left = a.units_left, rc_units_left = a.rc_units_left;
  uint32_t rc_nsplit = a.rc_nsplit, rc_ranges = a.rc_ranges, rc_msplits = a.rc_msplits, rc_gq = a.rc_gq, rc_H = a.rc_H;
  int nsplit = a.nsplit, ranges = a.ranges, share_bits = a.share_bits, msplits = a.msplits, gq = a.gq, H = a.H, KVBH = a.KVBH, S = a.S, M = a.M;
  asm("" : "+s"(upl), "+s"(rc_upl), "+s"(eights), "+s"(left), "+s"(rc_left), "+s"(whole_eights), "+s"(units_left),
           "+s"(rc_units_left), "+s"(spin), "+s"(ranges), "+s"(rc_ranges), "+s"(share_bits));
  asm("" : "+s"(rc_nsplit), "+s"(rc_msplits), "+s"(rc_gq), "+s"(rc_H), "+s"(nsplit), "+s"(msplits),
           "+s"(gq), "+s"(H), "+s"(KVBH), "+s"(S), "+s"(M) : "s"(a.words), "s"(a.anc), "s"(a.seq_len), "s"(a.scale_log2));
  // (units by eights, a unit's blocks 8 apart: on one XCD; what is left of them one key range after the other)
  const uint32_t octet = blockIdx.x >> 3, oct_unit = div_rc(octet, (uint32_t)nsplit, rc_nsplit);
  const uint32_t tail = blockIdx.x - whole_eights * (uint32_t)nsplit, tsplit = div_rc(tail, units_left, rc_units_left);
  const bool in_tail = blockIdx.x >= whole_eights * (uint32_t)nsplit;
  const uint32_t unit = in_tail ? whole_eights + tail - tsplit * units_left : oct_unit * 8 + (blockIdx.x & 7);
  const int split = (int)(in_tail ? tsplit : octet - oct_unit * (uint32_t)nsplit);
  const uint32_t lyr = div_rc(unit, upl, rc_upl);
  const uint32_t bid = unit - lyr * upl;
  const LayerPtrs& L = a.layer[lyr];
  // (the heads that are left, fewer than XCDs, take turns: a block of each, so that no XCD idles)
  const bool of_left = bid >= eights;
  const uint32_t rest = bid - eights, turn = div_rc(rest, left, rc_left);
  const uint32_t slot = of_left ? turn : bid >> 3;
  const uint32_t hq = div_rc(slot, (uint32_t)msplits, rc_msplits);
  const int ms = (int)(slot - hq * (uint32_t)msplits);
  const uint32_t kvq = of_left ? 0u : div_rc(hq, (uint32_t)gq, rc_gq), qg = hq - kvq * (uint32_t)gq;
  const int kvbh = (int)(of_left ? (uint32_t)KVBH - left + rest - turn * left : kvq * 8 + ((bid - lyr * spin) & 7));    // batch * Hkv + key/value head
  if (kvbh >= KVBH) return;                                 // (padding)
  const int bh = kvbh * gq + (int)qg;                       // batch * H + query head
  const int b = (int)div_rc((uint32_t)bh, (uint32_t)H, rc_H);
  const int m0 = ms * ROWS + rw * WROWS;       // first row of this wave
  int len = *(a.seq_len ? a.seq_len + b : reinterpret_cast<const int32_t*>(a.anc));          // (no lengths: something that can be read)
  asm("" : "+s"(len) : "s"(L.q), "s"(L.kc), "s"(L.vc), "s"(L.kt), "s"(L.vt));
  const int seq = a.seq_len ? min(max(len, 0), S) : S;
  const int GC = (seq + 31) >> 5, GT = (M + 31) >> 5, G = GC + GT;
  const int range = split >> share_bits, waves = KW << share_bits, wave_no = (split - (range << share_bits)) * KW + kw;
  // (beyond 2^32 / ranges, a few million keys, a bound may come out one group up, for both ranges that it parts; the last one, G, not)
  const int gbeg = (int)div_rc((uint32_t)(range * G), (uint32_t)ranges, rc_ranges);
  const int gend = (int)div_rc((uint32_t)((range + 1) * G), (uint32_t)ranges, rc_ranges);
  const uint16_t* kc = reinterpret_cast<const uint16_t*>(L.kc) + (int64_t)kvbh * S * DH;
  const uint16_t* vc = reinterpret_cast<const uint16_t*>(L.vc) + (int64_t)kvbh * S * DH;
  const uint16_t* kt = reinterpret_cast<const uint16_t*>(L.kt) + (int64_t)kvbh * M * DH;
  const uint16_t* vt = reinterpret_cast<const uint16_t*>(L.vt) + (int64_t)kvbh * M * DH;
  const uint16_t* qh = reinterpret_cast<const uint16_t*>(L.q) + (int64_t)bh * M * DH;
  float* const out = reinterpret_cast<float*>(L.out);

  // Key groups [0, GF) lie wholly inside the cache: no mask, no bounds.  The others (the ragged
  // end of the cache and the tree keys) go through the general path after them.
  const int GF = seq >> 5;
  // (in bytes, 32 bits: offsets to a wave-uniform pointer)
  const uint32_t koff = (uint32_t)(l16 * DH + g4 * 8) * 2;                  // my K chunk inside a group
  const uint32_t voff = (uint32_t)lane * 16;                                // my V chunks: + p * 64 chunks
  auto load_full = [&](Stage<DH>& st, int g) {
    const char* Kp = reinterpret_cast<const char*>(kc + (int64_t)g * (32 * DH));
    const char* Vp = reinterpret_cast<const char*>(vc + (int64_t)g * (32 * DH));
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        st.ka[t][ks] = __builtin_bit_cast(bf16x8, ld16(Kp + koff + (t * 32 * DH + ks * 64)));
#pragma unroll
    for (int p = 0; p < VCH; ++p) st.vr[p] = ld16(Vp + voff + p * 1024);
  };
  // general path: every load is unconditional and in bounds (row index clamped); absent keys are
  // masked out of the scores, and their V rows are zeroed on the way into LDS
  auto load_any = [&](Stage<DH>& st, int g) {
    const bool is_tree = g >= GC;
    const int kbase = is_tree ? (g - GC) * 32 : g * 32;
    const int last = (is_tree ? M : seq) - 1;
    const uint16_t* Kp = is_tree ? kt : kc;
    const uint16_t* Vp = is_tree ? vt : vc;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int row = min(kbase + t * 16 + l16, last);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        st.ka[t][ks] = __builtin_bit_cast(bf16x8, ld16(reinterpret_cast<const char*>(Kp) + ((uint32_t)row * (DH * 2) + g4 * 16) + ks * 64));
    }
#pragma unroll
    for (int p = 0; p < VCH; ++p) {
      const int c = lane + 64 * p;
      const int row = min(kbase + c / CPR, last);
      st.vr[p] = ld16(reinterpret_cast<const char*>(Vp) + ((uint32_t)row * (DH * 2) + (c % CPR) * 16));
    }
  };

  // Q as the B operand: column = tree row, 8 consecutive Dh per lane and step
  bf16x8 qb[NT][KS];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int m = min(m0 + nt * 16 + l16, M - 1);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qb[nt][ks] = __builtin_bit_cast(bf16x8, ld16(reinterpret_cast<const char*>(qh) + ((uint32_t)m * (DH * 2) + g4 * 16) + ks * 64));
  }

  f32x4 oacc[DT][NT], lacc[NT];
  float m_ref[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    m_ref[nt] = kMasked;
    lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const uint32_t one2 = 0x3F803F80u;   // two bf16 ones
  const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(one2, one2, one2, one2));

  unsigned char* vtile = smem + wave * (2 * VTILE);
  int buf = 0;
  const uint32_t vst = (uint32_t)((lane / CPR) * VPITCH + (lane % CPR) * 16);           // where my V chunks go
  const uint32_t vld = (uint32_t)((4 * g4 + (l16 >> 2)) * VPITCH + 8 * (l16 & 3));     // what I point the transposing read at

  // Which of the 32 keys of group g row m0 + nt 16 + l16 may see: the ancestor mask for tree
  // keys, the valid length for the ragged end of the cache.  The mask words are fetched here and
  // only looked at inside compute_group, so that the fetch does not hold up what follows.
  auto visibility = [&](uint64_t (&vis)[NT], int g) {
    const bool is_tree = g >= GC;
    const int kbase = is_tree ? (g - GC) * 32 : 0;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int m = min(m0 + nt * 16 + l16, M - 1);   // (rows past M are never written out)
      vis[nt] = a.anc[m * a.words + (kbase >> 6)];     // (a valid word also for cache groups: unused there)
    }
  };

  // One key group.  FULL (compile time): all 32 keys present and visible to every row.  Of the wave's tiles the first NL.
  auto compute_group = [&](const Stage<DH>& st, int g, const uint64_t (&vis)[NT], auto full_tag, auto live_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    constexpr int NL = decltype(live_tag)::value;
    const bool is_tree = g >= GC;
    const int kbase = is_tree ? (g - GC) * 32 : g * 32;
    const int limit = is_tree ? M : seq;                       // keys [kbase, limit) exist

    // S^T = K Q^T
    f32x4 sacc[2][NL];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int nt = 0; nt < NL; ++nt) {
        sacc[t][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          sacc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.ka[t][ks], qb[nt][ks], sacc[t][nt], 0, 0, 0);
      }

    // V rows into this wave's LDS tile, as they are
    unsigned char* tile = vtile + buf * VTILE;
#pragma unroll
    for (int p = 0; p < VCH; ++p) {
      uint4 v = st.vr[p];
      if (!FULL && kbase + (lane + 64 * p) / CPR >= limit) v = make_uint4(0, 0, 0, 0);   // absent keys: exact zeros
      *reinterpret_cast<uint4*>(tile + vst + p * (64 / CPR) * VPITCH) = v;
    }

    // softmax weights of the group; lane holds keys t*16 + 4*g4 + r of column l16
    uint32_t bits[NL];
    float mxl[NL];
    bool need = false;
#pragma unroll
    for (int nt = 0; nt < NL; ++nt) {
      bits[nt] = 0xFFFFFFFFu;
      if (!FULL) {
        const int left = seq - kbase;
        const uint32_t cache_bits = left >= 32 ? 0xFFFFFFFFu : ((1u << left) - 1u);
        bits[nt] = is_tree ? (uint32_t)(vis[nt] >> (kbase & 63)) : cache_bits;
        bits[nt] >>= 4 * g4;        // bit 16 t + r is now my key (t, r)
      }
      float v = kMasked;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float sc = sacc[t][nt][r];
          if (!FULL && !((bits[nt] >> (16 * t + r)) & 1u)) sc = kMasked;
          v = fmaxf(v, sc);
        }
      mxl[nt] = v > 0.5f * kMasked ? v * a.scale_log2 : kMasked;   // (scale > 0: the maximum commutes with it)
      need = need || (mxl[nt] > m_ref[nt] + kLazy);
    }
    if (__ballot(need)) {   // some row's reference moves: rare after a wave's first group
#pragma unroll
      for (int nt = 0; nt < NL; ++nt) {
        float v = mxl[nt];
        v = fmaxf(v, __shfl_xor(v, 16));
        v = fmaxf(v, __shfl_xor(v, 32));
        const bool up = v > m_ref[nt] + kLazy;               // decided per row: no row depends on another's scores
        const float nm = up ? v : m_ref[nt];
        const float alpha = __builtin_amdgcn_exp2f(m_ref[nt] - nm);
        m_ref[nt] = nm;
        lacc[nt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) oacc[dt][nt] *= alpha;
      }
    }
    bf16x8 pb[NL];
#pragma unroll
    for (int nt = 0; nt < NL; ++nt) {
      uint32_t pk[4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[t][nt][r], a.scale_log2, -m_ref[nt]));
          float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[t][nt][r + 1], a.scale_log2, -m_ref[nt]));
          if (!FULL) {
            if (!((bits[nt] >> (16 * t + r)) & 1u)) p0 = 0.f;
            if (!((bits[nt] >> (16 * t + r + 1)) & 1u)) p1 = 0.f;
          }
          pk[t * 2 + r / 2] = pack_bf16(p0, p1);
        }
      pb[nt] = __builtin_bit_cast(bf16x8, make_uint4(pk[0], pk[1], pk[2], pk[3]));
      lacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[nt], lacc[nt], 0, 0, 0);
    }

    // O^T += V^T P^T.  Contraction slot (g4, j) is key (j < 4 ? 0 : 16) + 4 g4 + j % 4 on both sides.
    // The transposing read hands lane (l16, g4) the four values V[key 4 g4 + j][dt 16 + l16]: within a
    // group of 16 lanes, lane s points at 4 consecutive Dh of key 4 g4 + s / 4 at Dh offset 4 (s % 4).
    wave_lds_sync();
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const unsigned char* src = tile + vld + dt * 32;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (s16x4 __attribute__((address_space(3)))*)(const __attribute__((address_space(3))) unsigned char*)src);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (s16x4 __attribute__((address_space(3)))*)(const __attribute__((address_space(3))) unsigned char*)(src + 16 * VPITCH));
      const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
      const bf16x8 va = __builtin_bit_cast(bf16x8, make_uint4(l2.x, l2.y, h2.x, h2.y));
#pragma unroll
      for (int nt = 0; nt < NL; ++nt)
        oacc[dt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb[nt], oacc[dt][nt], 0, 0, 0);
    }
    buf ^= 1;   // the next group writes the other tile while these reads may still be in flight
  };
  const std::integral_constant<bool, true> kFull;
  const std::integral_constant<bool, false> kAny;

  // ---- this wave's groups.  The full groups go through a ring of D stages: the loads of the next
  // D - 1 groups are in flight while one is worked on, and a stage is refilled as soon as it has
  // been consumed.  The wave's first general group is fetched before them and worked on while
  // the ring's first loads are in flight.
  auto run = [&](auto live) {
    const int h1 = min(gend, GF);                     // full groups: [gbeg, h1)
    const int c0 = max(gbeg, GF);                     // general groups: [c0, gend)
    const uint64_t novis[NT] = {};
    Stage<DH> cst;
    uint64_t vis[NT];
    int gx = c0 + wave_no;                               // next general group of this wave
    if (GF >= 1) {
      constexpr int D = 2;   // (deeper rings were no faster on long caches and slower on short ones: the
                             //  eight waves of a block already have sixteen groups in flight)
      Stage<DH> st[D];
      const bool pre = gx < gend;
      if (pre) { visibility(vis, gx); load_any(cst, gx); }
      // Ring loads are issued unconditionally (a group index past the end is clamped: a re-read
      // that is never used), so that the number of loads in flight is the same on every path and
      // each wait lets the younger loads stay in flight.
      int g = gbeg + wave_no;
      const int hl = max(h1 - 1, 0);
#pragma unroll
      for (int d = 0; d < D; ++d)
        if (!kLean || d < D - 1) load_full(st[d], min(g + d * waves, hl));
      if (pre) { compute_group(cst, gx, vis, kAny, live); gx += waves; }   // while the ring's loads are in flight
      if (kLean) load_full(st[D - 1], min(g + (D - 1) * waves, hl));
      // whole rounds of the ring, as long as at least the round's first refill is a group of this
      // wave (a round that would refill nothing is left to the tail below: a wave with D groups or
      // fewer would else spend half of the compute unit's load issue on re-reads nobody uses)
      while (g + D * waves < h1) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          compute_group(st[d], g, novis, kFull, live);
          load_full(st[d], min(g + D * waves, hl));
          g += waves;
        }
      }
#pragma unroll
      for (int d = 0; d < D; ++d) {               // what is left: up to D groups, already loaded
        if (g < h1) compute_group(st[d], g, novis, kFull, live);
        g += waves;
      }
    }
    for (; gx < gend; gx += waves) {                 // further general groups: rare, not pipelined
      visibility(vis, gx);
      load_any(cst, gx);
      compute_group(cst, gx, vis, kAny, live);
    }
  };
  // (a block behind an odd number of tiles has none in its last place: 129 rows as 5 + 4)
  if (NT >= 5 && m0 + (NT - 1) * 16 >= M) run(std::integral_constant<int, (NT > 1 ? NT - 1 : 1)>());
  else run(std::integral_constant<int, NT>());

  // ---- merge the waves of the block (fixed order => run-to-run identical): every wave brings
  // its O to the block's reference maximum and parks it in LDS; the sum over the waves is taken
  // on the way out
  // (the maxima and sums have a place of their own behind the V tiles, so a wave can leave them
  // there as soon as it is done; O is parked over the V tiles once every wave is done with them)
  constexpr int OBYTES = MS * ROWS * OPITCH * 4, VBYTES = KW * 2 * VTILE;
  float* s_o = reinterpret_cast<float*>(smem);                  // [MS][ROWS][OPITCH]
  float* s_m = reinterpret_cast<float*>(smem + (OBYTES > VBYTES ? OBYTES : VBYTES));   // [W][ROWS], then the block's: [ROWS]
  float* s_l = s_m + (W + 1) * ROWS;                            // [W][ROWS], then the block's: [ROWS]
  const int r0 = rw * WROWS;                                    // my first row inside the block
  if (g4 == 0) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      s_m[wave * ROWS + r0 + nt * 16 + l16] = m_ref[nt];
      s_l[wave * ROWS + r0 + nt * 16 + l16] = lacc[nt][0];
    }
  }
  __syncthreads();   // every wave is done with its V tiles too
  float fscale[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int col = r0 + nt * 16 + l16;
    float mm = kMasked;
#pragma unroll
    for (int w = 0; w < KW; ++w) mm = fmaxf(mm, s_m[(rw * KW + w) * ROWS + col]);
    float ll = 0.f;
#pragma unroll
    for (int w = 0; w < KW; ++w)
      ll += __builtin_amdgcn_exp2f(s_m[(rw * KW + w) * ROWS + col] - mm) * s_l[(rw * KW + w) * ROWS + col];
    fscale[nt] = __builtin_amdgcn_exp2f(m_ref[nt] - mm);
    if (kw == 0 && g4 == 0) { s_m[W * ROWS + col] = mm; s_l[W * ROWS + col] = ll; }
  }
  // MS slots of [ROWS][OPITCH] floats: with fewer slots than waves the upper waves park first and
  // the lower ones add themselves on top
#pragma unroll
  for (int round = (MS == KW ? 1 : 0); round < 2; ++round) {
    if (round == 1 && MS != KW) __syncthreads();
    const bool mine = round == 0 ? kw >= MS : kw < MS;
    if (mine) {
      const int sl = kw % MS;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int col = r0 + nt * 16 + l16;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          float4* dst = reinterpret_cast<float4*>(&s_o[(sl * ROWS + col) * OPITCH + dt * 16 + 4 * g4]);
          float4 v = make_float4(oacc[dt][nt][0] * fscale[nt], oacc[dt][nt][1] * fscale[nt],
                                 oacc[dt][nt][2] * fscale[nt], oacc[dt][nt][3] * fscale[nt]);
          if (round == 1 && MS != KW) { const float4 o = *dst; v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w; }
          *dst = v;
        }
      }
    }
  }
  __syncthreads();

  // ---- write: final rows if this block saw every key, else an unnormalised partial
  constexpr int C4 = DH / 4;
  const int mb = ms * ROWS;                                     // first row of the block
  // first row of the unit's partials, where there are any (the launch then has a few hundred blocks)
  const uint32_t part0 = (lyr * (uint32_t)(KVBH * gq) + (uint32_t)bh) * (uint32_t)(nsplit * a.rows_pad) + (uint32_t)mb;
  const __amdgpu_buffer_rsrc_t dev_o = device_buffer(a.ws_o, a.ws_o_bytes), dev_ml = device_buffer(a.ws_ml, a.ws_ml_bytes);
  for (int idx = threadIdx.x; idx < ROWS * C4; idx += W * 64) {
    const int r = idx / C4, c4 = idx % C4;
    const int m = mb + r;
    if (m >= M) continue;
    float4 v = *reinterpret_cast<const float4*>(&s_o[r * OPITCH + c4 * 4]);
#pragma unroll
    for (int w = 1; w < MS; ++w) {
      const float4 o = *reinterpret_cast<const float4*>(&s_o[(w * ROWS + r) * OPITCH + c4 * 4]);
      v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
    }
    const float bm = s_m[W * ROWS + r], bl = s_l[W * ROWS + r];
    if (nsplit == 1) {
      const float inv = 1.0f / bl;
      v.x *= inv; v.y *= inv; v.z *= inv; v.w *= inv;
      store_out4(out, a.out_bf16 != 0, ((int64_t)bh * M + m) * DH + c4 * 4, v);
    } else {   // read by another block of this launch: stores that are visible device-wide when they complete
      const uint32_t prow = part0 + (uint32_t)(split * a.rows_pad + r);
      store_dev(dev_o, (uint32_t)((prow * DH + c4 * 4) * 4), v);
      if (c4 == 0) store_dev(dev_ml, (uint32_t)(prow * 8), make_float2(bm, bl));
    }
  }
  if (nsplit == 1) return;

  // ---- the block of this (head, row range) that finishes last adds the splits up, in split order
  // Every wave first waits until its own stores of the partial have completed (a device-scope
  // store is visible to every compute unit once it has completed; the workgroup barrier alone
  // waits for LDS traffic only), then the barrier gathers the waves, and only then the ticket is
  // taken.  The ticket and the reads below are device-scope atomics as well, so no cache
  // write-back or invalidate is needed.
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __syncthreads();
  if (threadIdx.x == 0)
    s_ticket = __hip_atomic_fetch_add(&a.counters[unit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (s_ticket != nsplit - 1) return;
  for (int idx = threadIdx.x; idx < ROWS * C4; idx += W * 64) {
    const int r = idx / C4, c4 = idx % C4;
    const int m = mb + r;
    if (m >= M) continue;
    // (four splits at a time: all their loads are in flight together)
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float ll = 0.f, mm = kMasked;
    for (int s0 = 0; s0 < nsplit; s0 += 4) {
      float2 ml[4];
      float4 o[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t prow = part0 + (uint32_t)(min(s0 + u, nsplit - 1) * a.rows_pad + r);    // (a split past the end: read again, weight 0)
        ml[u] = load_dev2(dev_ml, (uint32_t)(prow * 8));
        o[u] = load_dev4(dev_o, (uint32_t)((prow * DH + c4 * 4) * 4));
      }
      float nm = mm;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s0 + u < nsplit) nm = fmaxf(nm, ml[u].x);
      const float keep = __builtin_amdgcn_exp2f(mm - nm);       // (the first batch: exp2(-huge) = 0 on zeros)
      acc.x *= keep; acc.y *= keep; acc.z *= keep; acc.w *= keep; ll *= keep;
      mm = nm;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float f = s0 + u < nsplit ? __builtin_amdgcn_exp2f(ml[u].x - mm) : 0.f;
        ll += f * ml[u].y;
        acc.x += f * o[u].x; acc.y += f * o[u].y; acc.z += f * o[u].z; acc.w += f * o[u].w;
      }
    }
    const float inv = 1.0f / ll;
    store_out4(out, a.out_bf16 != 0, ((int64_t)bh * M + m) * DH + c4 * 4,
               make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv));
  }
  if (threadIdx.x == 0)   // ready for the next call
    __hip_atomic_store(&a.counters[unit], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- fp32 path
struct AttnArgsF32 {
  const int32_t* seq_len; const uint64_t* anc;
  int32_t B, H, Hkv, S, M, words;
  int32_t mtiles, gq, out_bf16;     // row tiles; query heads per key/value head; out holds bf16 instead of float
  float scale;
  int32_t nsplit;                   // key ranges per (batch, head), and with more than one their partials:
  uint32_t rc_nsplit, rc_per, rc_mtiles, rc_Hkv;   // reciprocals (div_rc) of nsplit, mtiles * gq, mtiles and Hkv
  LayerPtrs layer[kLayersPerLaunch];     // blockIdx.y picks the layer
  float4* ws_o;                     // [layer][BH][mtiles][nsplit][16][Dh]  unnormalised partial O
  float2* ws_ml;                    // [layer][BH][mtiles][nsplit][16]      (reference max, sum)
};

// e^t for t <= 0 (0 below -200, NaN stays): the hardware's 2^x on t log2 e, whose rounding is taken back to first
// order.  Without that, scores of a few units cost a fifth of the accuracy; expf keeps it, but its registers
// spill in the kernel (12 bytes a lane at rows of 64).
__device__ __forceinline__ float exp_neg(float t) {
  constexpr float kLog2e = 1.44269504088896340736f, kLn2 = 0.69314718055994530942f;
  t = t < -200.f ? -200.f : t;
  const float x = t * kLog2e, r = __builtin_amdgcn_exp2f(x);
  return __builtin_fmaf(r, __builtin_fmaf(t, kLog2e, -x) * kLn2, r);
}

// One tile of 16 keys in flight.  K: lane (i, g) holds of key i the dimensions 16 t + 4 g .. + 3; V: of keys
// 4 g + r the dimensions 64 h + 4 i .. + 3 (i = lane % 16, g = lane / 16).
template <int DH>
struct StageF32 {
  f32x4 k[DH / 16];
  f32x4 v[4][DH / 64];
};

// Rows of K and V by position: the cache first, then the tree.
template <int DH>
struct KeysF32 {
  const float* kc; const float* vc; const float* kt; const float* vt;
  int seq, n;
  __device__ __forceinline__ const float* k(int j) const { return j < seq ? kc + (int64_t)j * DH : kt + (int64_t)(j - seq) * DH; }
  __device__ __forceinline__ const float* v(int j) const { return j < seq ? vc + (int64_t)j * DH : vt + (int64_t)(j - seq) * DH; }
  __device__ __forceinline__ void load(StageF32<DH>& st, int tile, int lane) const {
    const int i = lane & 15, g = lane >> 4;
    const float* kr = k(min(tile * 16 + i, n - 1));          // (past the end: the last key again, masked below)
#pragma unroll
    for (int t = 0; t < DH / 16; ++t) st.k[t] = *reinterpret_cast<const f32x4*>(kr + 16 * t + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* vr = v(min(tile * 16 + 4 * g + r, n - 1));
#pragma unroll
      for (int h = 0; h < DH / 64; ++h) st.v[r][h] = *reinterpret_cast<const f32x4*>(vr + 64 * h + 4 * i);
    }
  }
};

__device__ __forceinline__ void fma4(float4& o, float f, float4 x) {
  o.x = __builtin_fmaf(f, x.x, o.x); o.y = __builtin_fmaf(f, x.y, o.y);
  o.z = __builtin_fmaf(f, x.z, o.z); o.w = __builtin_fmaf(f, x.w, o.w);
}

// What a block works on: a tile of 16 rows of one (batch, head).  `n` counts the tiles of the block's XCD: the
// blocks of a key/value head sit on one XCD (block index mod 8) and share its L2.
template <int DH>
struct CellF32 {
  KeysF32<DH> keys;
  const float* q;                   // the (batch, head)'s queries
  float* out;
  int64_t cell, e0;                 // number of the tile over all layers; first element of its output
  int tile0;
  bool live;
  // (As in the bf16 kernel: every argument and the layer's pointers are asked for at once, and reciprocals instead of divisions:
  // 4 heads, 16 rows, 256 keys 10.0 -> 9.6 us.)
  // parts: blocks per tile (key ranges); part: the block's
  __device__ __forceinline__ CellF32(const AttnArgsF32& a, bool parts, int& part) {
    const LayerPtrs& L = a.layer[blockIdx.y];
    uint32_t mtiles = (uint32_t)a.mtiles, rc_nsplit = a.rc_nsplit, rc_per = a.rc_per, rc_mtiles = a.rc_mtiles, rc_Hkv = a.rc_Hkv;
    asm("" : "+s"(mtiles), "+s"(rc_nsplit), "+s"(rc_per), "+s"(rc_mtiles), "+s"(rc_Hkv)
        : "s"(a.seq_len), "s"(a.anc), "s"(a.B), "s"(a.H), "s"(a.Hkv), "s"(a.S), "s"(a.M), "s"(a.words), "s"(a.gq), "s"(a.scale),
          "s"(a.nsplit), "s"(L.q), "s"(L.kc), "s"(L.vc), "s"(L.kt), "s"(L.vt));
    uint32_t n = blockIdx.x >> 3;
    part = 0;
    if (parts) {
      const uint32_t t = div_or_rc(n, (uint32_t)a.nsplit, rc_nsplit);
      part = (int)(n - t * (uint32_t)a.nsplit);
      n = t;
    }
    const uint32_t per = mtiles * (uint32_t)a.gq, heads = div_or_rc(n, per, rc_per), rest = n - heads * per;
    const int kvbh = (int)heads * 8 + (int)(blockIdx.x & 7);
    live = kvbh < a.B * a.Hkv;
    if (!live) return;
    const uint32_t qg = div_or_rc(rest, mtiles, rc_mtiles);
    const int bh = kvbh * a.gq + (int)qg, b = (int)div_or_rc((uint32_t)kvbh, (uint32_t)a.Hkv, rc_Hkv);
    tile0 = (int)(rest - qg * mtiles);
    cell = ((int64_t)blockIdx.y * a.B * a.H + bh) * (int)mtiles + tile0;
    e0 = ((int64_t)bh * a.M + tile0 * 16) * DH;
    keys.kc = reinterpret_cast<const float*>(L.kc) + (int64_t)kvbh * a.S * DH;
    keys.vc = reinterpret_cast<const float*>(L.vc) + (int64_t)kvbh * a.S * DH;
    keys.kt = reinterpret_cast<const float*>(L.kt) + (int64_t)kvbh * a.M * DH;
    keys.vt = reinterpret_cast<const float*>(L.vt) + (int64_t)kvbh * a.M * DH;
    keys.seq = a.seq_len ? min(max(a.seq_len[b], 0), a.S) : a.S;
    keys.n = keys.seq + a.M;
    q = reinterpret_cast<const float*>(L.q) + (int64_t)bh * a.M * DH;
    out = reinterpret_cast<float*>(L.out);
  }
};

// Scores of a tile: lane (i, g) holds those of tree row i with keys 4 g + r, -inf where the row does not see the key.
// row: that tree row.
template <int DH>
__device__ __forceinline__ void f32_scores(const AttnArgsF32& a, const StageF32<DH>& st, const f32x4 (&q)[DH / 16], int tile,
                                           int row, int g, int seq, float (&sc)[4]) {
  f32x4 s = {0.f, 0.f, 0.f, 0.f};      // four chains of Dh / 4 products, two at a time
#pragma unroll
  for (int t0 = 0; t0 < DH / 16; t0 += DH / 32) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = t0; t < t0 + DH / 32; t += 2)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(st.k[t][e], q[t][e], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(st.k[t + 1][e], q[t + 1][e], s1, 0, 0, 0);
      }
    s += s0 + s1;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) sc[r] = s[r] * a.scale;
  if (tile * 16 + 16 > seq) {                             // tree keys, or past the end
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = tile * 16 + 4 * g + r - seq;
      const uint64_t w = t >= 0 && t < a.M ? a.anc[(int64_t)row * a.words + (t >> 6)] >> (t & 63) : (uint64_t)(t < 0);
      if (!(w & 1ull)) sc[r] = -INFINITY;
    }
  }
}

// A wave's accumulators [4 HT] to the merge buffer's row (wave, i), row pitch P4.
template <int DH>
__device__ __forceinline__ void f32_park(float4* s_o, int P4, int wave, int lane, const f32x4 (&acc)[DH / 16]) {
  const int i = lane & 15, g = lane >> 4;
#pragma unroll
  for (int h = 0; h < DH / 64; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      s_o[(wave * 16 + i) * P4 + 16 * h + 4 * g + r] =
          make_float4(acc[4 * h][r], acc[4 * h + 1][r], acc[4 * h + 2][r], acc[4 * h + 3][r]);
}

// Divide by the row's sum and write; all threads of the block.  A key that a row does not see, or whose weight
// underflows, adds an exact 0 whatever its V row holds, which a product of matrices does not give: where a
// result is not finite the tile is done again, now with the rows' maxima (mm) known.  V is then multiplied with its
// infinities and NaN as zeros, and in tiles that hold any they are counted, by a product with "the key has a
// weight", and put where they belong.  One more pass over the keys, by one block per row tile (a second tile in
// flight gains nothing: a compute unit takes in what it can).  With a NaN in one V row, key by key in
// a block per row -> key by key in a wave per row -> so: 4 heads, 16 rows, 256 keys of 64: 13.3 -> 128 -> 17.8 us;
// 16 heads, 96 rows, 1898 keys: 197 -> 866 -> 56; 12 heads, 21 rows, 1498 keys of 128: 76 -> 1556 -> 65; 8 heads on 2
// shared ones, 27 rows, 1024 keys of 128: 46 -> 1075 -> 50.
template <int DH, int W>
__device__ __forceinline__ void f32_finish(const AttnArgsF32& a, const CellF32<DH>& c, float4* s_o, bool mine, int orow, int c4,
                                           float4 o, float mm, float ll) {
  constexpr int HT = DH / 64, P4 = DH / 4 + 1;
  __shared__ float s_mx[16], s_sum[W][16];
  __shared__ __align__(16) int s_again[W];
  const int tid = formed_anew(threadIdx.x);
  if (mine) { o.x /= ll; o.y /= ll; o.z /= ll; o.w /= ll; }
  const bool finite = isfinite(o.x) && isfinite(o.y) && isfinite(o.z) && isfinite(o.w);
  if (c4 == 0 && tid < 16 * DH / 4) s_mx[orow] = mm;
  const int odd_wave = __any(!finite) ? 1 : 0;
  if ((tid & 63) == 0) s_again[tid >> 6] = odd_wave;
  __syncthreads();
  int again = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) again |= s_again[w];
  if (__builtin_amdgcn_readfirstlane(again)) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
    const int row = min(c.tile0 * 16 + i, a.M - 1), all = (c.keys.n + 15) / 16;
    const float mx = s_mx[min(i, a.M - 1 - c.tile0 * 16)];
    f32x4 q[DH / 16], acc[4 * HT] = {};
#pragma unroll
    for (int t = 0; t < DH / 16; ++t) q[t] = *reinterpret_cast<const f32x4*>(c.q + (int64_t)row * DH + 16 * t + 4 * g);
    float l = 0.f;
    for (int tile = wave; tile < all; tile += W) {
      StageF32<DH> st;
      c.keys.load(st, tile, lane);
      float sc[4], has[4];
      f32_scores<DH>(a, st, q, tile, row, g, c.keys.seq, sc);
      bool odd = false;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc[r] = sc[r] == -INFINITY ? 0.f : exp_neg(sc[r] - mx);
        has[r] = sc[r] != 0.f ? 1.f : 0.f;
        l += sc[r];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < HT; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = st.v[r][h][e];
            odd = odd || !isfinite(v);
            acc[4 * h + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(isfinite(v) ? v : 0.f, sc[r], acc[4 * h + e], 0, 0, 0);
          }
      if (__any(odd)) {
#pragma unroll
        for (int h = 0; h < HT; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            f32x4 n = {0.f, 0.f, 0.f, 0.f};              // of the 16 keys: +inf count 1, -inf 32, NaN 33
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float v = st.v[r][h][e];
              const float count = isfinite(v) ? 0.f : (v > 0.f ? 1.f : (v < 0.f ? 32.f : 33.f));
              n = __builtin_amdgcn_mfma_f32_16x16x4f32(count, has[r], n, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int x = (int)n[r];
              if (x & 31) acc[4 * h + e][r] += INFINITY;
              if (x >> 5) acc[4 * h + e][r] -= INFINITY;              // (both: NaN)
            }
          }
      }
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (lane < 16) s_sum[wave][i] = l;
    f32_park<DH>(s_o, P4, wave, lane, acc);
    __syncthreads();
    if (mine && !finite) {
      o = make_float4(0.f, 0.f, 0.f, 0.f);
      ll = 0.f;
#pragma unroll 1
      for (int w = 0; w < W; ++w) {
        fma4(o, 1.f, s_o[(w * 16 + orow) * P4 + c4]);
        ll += s_sum[w][orow];
      }
      o.x /= ll; o.y /= ll; o.z /= ll; o.w /= ll;
    }
  }
  if (mine) store_out4(c.out, a.out_bf16 != 0, c.e0 + (int64_t)orow * DH + c4 * 4, o);
}

// A block is 16 tree rows of one (batch, head); its W waves take the 16-key tiles in turn, the loads of a
// wave's next tile issued before it works on the current one.  Both products run on the float32 matrix cores
// (16x16x4, float32 products and sums):
//   S^T[16 keys x 16 rows] = K Q^T     K and Q with the dimensions dealt so that a lane's operands are what
//                                      its 16-byte loads bring
//   O^T[Dh x 16 rows] += V^T P^T       the weights are already where the B operand wants them, V's dimensions
//                                      are dealt like K's: no LDS between the loads and the products
// Bound by the latency of a wave's few serial tiles at small shapes, by the matrix cores and L2 at large ones.
// A block per row with a key per thread, which this replaces, read every key once per row and its K rows 64
// cache lines at a time.  Before -> now: 4 heads, 16 rows, 256 keys of 64: 13.3 -> 10.3 us; 16 heads, 96 rows,
// 1898 keys of 64: 172 -> 25.5 us; 12 heads, 21 rows, 1498 keys of 128: 76 -> 20 us.  Error against 64 bits, mean
// of 12 inputs: 2.1e-7 -> 1.7e-7 at the first, 5.9e-7 -> 2.1e-7 at 4096 keys.
// Where the launch leaves compute units idle the keys of a (batch, head) are cut into ranges, a block each (one
// compute unit takes in some tens of bytes a nanosecond, whatever its waves ask for) and a second kernel adds
// the partials up in the order of the ranges.  (Not a ticket in the handle: calls of this type keep no state.)
template <int DH, int W>
__global__ __launch_bounds__(W * 64) void tree_attn_f32_kernel(AttnArgsF32 a) {
  constexpr int HT = DH / 64, P4 = DH / 4 + 1;              // row pitch of the merge buffer in float4
  static_assert(16 * DH / 4 == W * 64 / (W == 16 && DH == 64 ? 4 : 1), "an output piece per thread");
  extern __shared__ __align__(16) unsigned char s_f32[];
  float4* const s_o = reinterpret_cast<float4*>(s_f32);     // [W][16][P4]
  __shared__ float s_m[W][16], s_l[W][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  int split;
  const CellF32<DH> c(a, true, split);
  if (!c.live) return;
  const KeysF32<DH>& keys = c.keys;
  const int seq = keys.seq, M = a.M, tile0 = c.tile0;
  const int all = (keys.n + 15) / 16;
  const int tbeg = (int)div_or_rc((uint32_t)(split * all), (uint32_t)a.nsplit, a.rc_nsplit);
  const int tend = (int)div_or_rc((uint32_t)((split + 1) * all), (uint32_t)a.nsplit, a.rc_nsplit);
  const int row = min(tile0 * 16 + i, M - 1);               // (rows past the last: the last one again, not written)

  StageF32<DH> cur, nxt;
  if (tbeg + wave < tend) keys.load(cur, tbeg + wave, lane);
  f32x4 q[DH / 16];
#pragma unroll
  for (int t = 0; t < DH / 16; ++t) q[t] = *reinterpret_cast<const f32x4*>(c.q + (int64_t)row * DH + 16 * t + 4 * g);
  f32x4 acc[4 * HT] = {};
  float m = -INFINITY, l = 0.f;
  for (int tile = tbeg + wave; tile < tend; tile += W) {
    if (tile + W < tend) keys.load(nxt, tile + W, lane);
    float sc[4];
    f32_scores<DH>(a, cur, q, tile, row, g, seq, sc);
    float mn = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
    mn = fmaxf(mn, __shfl_xor(mn, 16));
    mn = fmaxf(mn, __shfl_xor(mn, 32));
    mn = fmaxf(mn, m);
    if (__any(mn != m)) {
      const float f = mn == m ? 1.f : exp_neg(m - mn);
      l *= f;
#pragma unroll
      for (int d = 0; d < 4 * HT; ++d) acc[d] *= f;
      m = mn;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sc[r] = sc[r] == -INFINITY ? 0.f : exp_neg(sc[r] - m);
      l += sc[r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[4 * h + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.v[r][h][e], sc[r], acc[4 * h + e], 0, 0, 0);
    cur = nxt;
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  const int tid2 = formed_anew(tid), lane2 = tid2 & 63;
  if (lane2 < 16) { s_m[wave][lane2] = m; s_l[wave][lane2] = l; }
  if (tbeg + wave < tend) f32_park<DH>(s_o, P4, wave, lane2, acc);
  __syncthreads();

  const int orow = tid2 / (DH / 4), c4 = tid2 % (DH / 4);
  const bool mine = tid2 < 16 * DH / 4 && tile0 * 16 + orow < M;
  const int nw = min(W, tend - tbeg);
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  float mm = -INFINITY, ll = 0.f;
  if (mine) {
    float mw[W], lw[W];                     // (a wave without a tile wrote -inf and 0)
#pragma unroll
    for (int w = 0; w < W; ++w) { mw[w] = s_m[w][orow]; lw[w] = s_l[w][orow]; }
#pragma unroll
    for (int w = 0; w < W; ++w) mm = fmaxf(mm, mw[w]);
    float4 o1 = o;                          // (the odd waves' sums)
    float l1 = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w)
      if (w < nw) {
        const float f = mw[w] == -INFINITY ? 0.f : exp_neg(mw[w] - mm);
        fma4(w & 1 ? o1 : o, f, s_o[(w * 16 + orow) * P4 + c4]);
        (w & 1 ? l1 : ll) = __builtin_fmaf(f, lw[w], w & 1 ? l1 : ll);
      }
    o.x += o1.x; o.y += o1.y; o.z += o1.z; o.w += o1.w;
    ll += l1;
  }
  if (a.nsplit > 1) {
    const int64_t prow = (c.cell * a.nsplit + split) * 16 + orow;
    if (mine) {
      a.ws_o[prow * (DH / 4) + c4] = o;
      if (c4 == 0) a.ws_ml[prow] = make_float2(mm, ll);
    }
    return;
  }
  f32_finish<DH, W>(a, c, s_o, mine, orow, c4, o, mm, ll);
}

// The partials of a row tile's key ranges, added up in their order: four floats of a row per thread.
template <int DH, int W>
__global__ __launch_bounds__(W * 64) void tree_attn_f32_merge_kernel(AttnArgsF32 a) {
  extern __shared__ __align__(16) unsigned char s_f32[];    // (for tiles that are done again)
  int none;
  const CellF32<DH> c(a, false, none);
  if (!c.live) return;
  const int tid = threadIdx.x, orow = tid / (DH / 4), c4 = tid % (DH / 4);
  const bool mine = tid < 16 * DH / 4 && c.tile0 * 16 + orow < a.M;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  float mm = -INFINITY, ll = 0.f;
  if (mine) {
    const int64_t p0 = c.cell * a.nsplit * 16 + orow;
    for (int u = 0; u < a.nsplit; ++u) mm = fmaxf(mm, a.ws_ml[p0 + 16 * u].x);
#pragma unroll 4
    for (int u = 0; u < a.nsplit; ++u) {
      const float2 ml = a.ws_ml[p0 + 16 * u];
      const float4 x = a.ws_o[(p0 + 16 * u) * (DH / 4) + c4];
      const float f = ml.x == -INFINITY ? 0.f : exp_neg(ml.x - mm);
      ll = __builtin_fmaf(f, ml.y, ll);
      fma4(o, f, x);
    }
  }
  f32_finish<DH, W>(a, c, reinterpret_cast<float4*>(s_f32), mine, orow, c4, o, mm, ll);
}

template <int DH, int W>
int32_t launch_f32(const AttnArgsF32& a, int n_layers, hipStream_t s) {
  static LppLdsLimit limit;
  auto kern = tree_attn_f32_kernel<DH, W>;
  const size_t lds = (size_t)W * 16 * (DH + 4) * sizeof(float);
  const int32_t st = lpp_ensure_lds(reinterpret_cast<const void*>(kern), limit, lds, 48 * 1024);
  if (st != LPP_OK) return st;
  const int64_t blocks = 8 * (((int64_t)a.B * a.Hkv + 7) / 8) * a.gq * a.mtiles * a.nsplit;
  if (blocks >= (1ll << 31)) return LPP_EUNSUPPORTED;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks, (unsigned)n_layers), dim3(W * 64), lds, s, a);
  LPP_HIP_TRY(hipGetLastError());
  if (a.nsplit > 1) {
    static LppLdsLimit merge_limit;
    auto merge = tree_attn_f32_merge_kernel<DH, W>;
    const int32_t mst = lpp_ensure_lds(reinterpret_cast<const void*>(merge), merge_limit, lds, 48 * 1024);
    if (mst != LPP_OK) return mst;
    hipLaunchKernelGGL(merge, dim3((unsigned)(blocks / a.nsplit), (unsigned)n_layers), dim3(W * 64), lds, s, a);
    LPP_HIP_TRY(hipGetLastError());
  }
  return LPP_OK;
}

// Key ranges per (batch, head) of the float32 kernel: only while a compute unit would idle, of kRangeF32 key tiles
// or more: a tile costs a block 0.2 us (rows of 64) or 0.4 us (128), the second kernel about 3 us, so that two
// ranges of 16 are the least that gain.  One range -> this rule, 4 heads: 512 keys 12.5 -> 11.7 and 20.9 -> 17.2
// us; 4096 keys 56 -> 14 and 106 -> 24 us (both sides before the exponential above, which adds about 1 us).
constexpr int kRangeF32 = 16;
// Keys of a row, at most: no need of the kernel's (it keeps no scores), but what lpp.h states and the tests cover.
constexpr int64_t kMostKeysF32 = 36864;
int f32_splits(const lpp_tree* tree, int B, int H, int S, int layers) {
  const int64_t blocks = (int64_t)B * H * ((tree->M + 15) / 16) * std::max(1, std::min(layers, kLayersPerLaunch));
  const int64_t tiles = ((int64_t)S + tree->M + 15) / 16;
  return (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(tree->n_cu / blocks, tiles / kRangeF32), 16));
}

// Bytes of its partials: [O | max, sum]; nothing for one range.
size_t f32_workspace(const lpp_tree* tree, int B, int H, int Dh, int layers, int nsplit, size_t* o_bytes) {
  if (nsplit < 2) return 0;
  const size_t rows = (size_t)B * H * ((tree->M + 15) / 16) * 16 * std::min(layers, kLayersPerLaunch) * nsplit;
  if (o_bytes) *o_bytes = rows * Dh * sizeof(float);
  return rows * (Dh + 2) * sizeof(float);
}

struct AttnPlan {
  int mtiles, nt, msplits;          // row tiles of 16, those of a wave, row ranges of a (batch, head)
  int ranges, share, kw;            // key ranges of a (batch, head), the blocks that share one, the waves of a block
  size_t lds;
};

// A block is one range of NT * 16 tree rows of one (batch, head) and one range of key groups;
// its KW waves take the key groups in turn.  The blocks of a head that differ in the row range
// read the same keys at about the same time and sit on the same XCD, so that the second read is
// served by its L2.  Key splits (which cost a pass through the workspace) are only added while
// the launch (all its layers) would leave compute units idle.
// How the keys fall to waves says where a row's weights, of which the largest of each wave's reference is exact, are rounded to
// bf16, and so how large the error is: 4 waves instead of 8, or instead of 24 in three ranges, make it 5 to 15 % larger against
// float64 (scores of unit spread), 25 to 60 % with four times the scores.  Hence two parts: the waves and ranges of a
// (batch, head), by the blocks that two or more tiles a wave would make; then which of these waves, and which rows, share a block.  That
// only changes time (and the order of the float32 sums over waves).
AttnPlan plan_attention(const lpp_tree* tree, int B, int H, int S, int Dh, int layers, bool may_share = true) {
  AttnPlan p;
  p.mtiles = (tree->M + 15) / 16;
  const int GT = (tree->M + 31) / 32, G = (S + 31) / 32 + GT;
  const int64_t n_cu = tree->n_cu, heads = (int64_t)B * H * std::max(1, std::min(layers, kLayersPerLaunch));
  // ---- how the keys fall to waves: `ranges` of them, of 4 or 8 waves each
  // Up to 64 rows: two tiles per wave and one or two blocks per head (enough blocks to fill the
  // chip at small batch).  More rows: up to five tiles per wave, so that as few blocks as possible
  // stream the same K/V out of L2.
  if (p.mtiles <= 4 || Dh != 64) {
    p.nt = p.mtiles == 1 ? 1 : 2;
    p.msplits = (p.mtiles + p.nt - 1) / p.nt;
    // Few heads (a quarter of the compute units or fewer would get a block): one tile per wave and
    // twice the row ranges fill the chip with blocks that need no more key splits than before.
    // (Head size 64 only: measured slower at 128, where a one-tile wave holds as many registers.)
    if (Dh == 64 && p.nt == 2 && heads * p.msplits * 4 <= n_cu) {
      p.nt = 1;
      p.msplits = p.mtiles;
    }
  } else {
    p.msplits = (p.mtiles + 4) / 5;
    p.nt = (p.mtiles + p.msplits - 1) / p.msplits;
  }
  const int64_t blocks_bh = heads * p.msplits;
  // Ranges of 8 waves, a block on a compute unit -- unless the launch has more blocks than compute units
  // and a wave of a 4-wave block still has two groups or more: then two or three such blocks share
  // a compute unit and cover each other's fixed latencies (first bytes, in-block merge, write-out)
  // and stalls, which the waves of one block, in step with each other, cannot.  With three tiles or
  // more per wave (two waves per SIMD either way) that pays from two rounds of blocks on.
  const int waves = G >= 8 && ((p.nt == 2 && blocks_bh > n_cu) || (p.nt >= 3 && Dh == 64 && blocks_bh >= 2 * n_cu)) ? 4 : 8;
  // key splits only while a compute unit would idle, at least two key groups per wave
  p.ranges = (int)std::max<int64_t>(1, std::min<int64_t>(n_cu / blocks_bh, G / (2 * waves)));

  // ---- the blocks
  p.kw = waves;
  p.share = 1;
  // Launches of few blocks, which latency bounds (first bytes, in-block merge, merge of key ranges): a block costs what its waves
  // have to merge, 4 to 16 KB of sums each, and what it reads.  One tile a wave, then two, while the blocks are no more than the
  // compute units and these take in no more than 330 KB (660 KB) of keys and values on average.  Over 220 shapes (up to 256 heads,
  // 9 to 129 rows, 64 to 4096 keys), with the rule for shared ranges, launches take 1.01 times the best of all such choices and 0.92 of
  // what they take without the two, none of them more: 4 heads of 64, 100 rows, 1313 keys 15.3 -> 7.6 us; 40 heads, 121 rows, 1914 keys
  // 26.1 -> 16.4; 4 heads of 128, 27 rows, 1621 keys 13.8 -> 10.1.
  const int weight = Dh / 64;                     // a group of 32 keys and values: 8 KB each
  for (int nt = 1; nt <= 2 && nt < p.nt; ++nt) {
    const int64_t units = heads * ((p.mtiles + nt - 1) / nt);
    if (units * p.ranges > n_cu || units * G * weight > 40 * nt * n_cu) continue;
    p.nt = nt;
    p.msplits = (p.mtiles + nt - 1) / nt;
  }
  // Ranges of 8 waves in two blocks of 4, which merge less each, while every compute unit has one at most: 16 heads, 27 rows, 1024 keys
  // 8.6 -> 7.3 us.  (From five ranges on the merge of twice as many costs more: 20 heads, 11 rows, 4075 keys 9.7 -> 10.5 us.)
  if (waves == 8 && may_share && p.ranges >= 2 && p.ranges <= 4 && heads * p.msplits * p.ranges * 2 <= n_cu) {
    p.kw = 4;
    p.share = 2;
  }
  // Full groups and the others are each dealt from the first wave on: with four of each at most, waves 5 to 8 have none.
  // Without them a compute unit holds more than one block: 512 heads, 24 rows, 77 keys, 4 layers 44.1 -> 22.6 us; 60 heads, 31 rows, 100 keys 6.1 -> 5.1.
  if (S / 32 <= 4 && GT <= 3) p.kw = 4;
  // 33 to 64 rows in blocks of 4 waves: all of them in one block, so that K/V leave L2 once: 16 layers of 4 items x 24 heads, 61 rows,
  // 1024 keys 86.8 -> 75.5 us, 8 layers 52.5 -> 46.5.  Four tiles a wave only from 24 groups on (160 heads, 52 rows, 246 keys 9.1 -> 10.0
  // us; 576 heads, 19 groups 8 % more, 1024 heads, 31 groups 13 % less), and not where
  // they end in a second round that is short (61 rows, 1024 keys, 288 heads 19.9 -> 22.1 us, 384 heads 20.3 -> 23.1; 480 heads 29.7 -> 25.7).
  if (Dh == 64 && p.mtiles >= 3 && p.nt == 2 && waves == 4 &&
      (p.mtiles == 3 || G >= 48 || (G >= 24 && (heads <= n_cu || heads * 4 >= n_cu * 7)))) {
    p.nt = p.mtiles;
    p.msplits = 1;
  }
  const int rows = p.nt * 16;
  const size_t vt = (size_t)p.kw * 2 * 32 * (Dh * 2 + 32);
  const int ms = (size_t)p.kw * rows * (Dh + 4) * 4 <= std::max<size_t>(vt, (size_t)p.kw * 12 * 1024) ? p.kw : p.kw / 2;
  const size_t og = (size_t)ms * rows * (Dh + 4) * sizeof(float);
  p.lds = (vt > og ? vt : og) + (size_t)2 * (p.kw + 1) * rows * sizeof(float);
  return p;
}

template <int DH, int NT, int RW, int KW>
int32_t launch_bf16(const AttnArgs& a, const AttnPlan& p, int64_t blocks, hipStream_t s) {
  static LppLdsLimit limit;
  auto kern = tree_attn_bf16_kernel<DH, NT, RW, KW>;
  const int32_t st = lpp_ensure_lds(reinterpret_cast<const void*>(kern), limit, p.lds, 48 * 1024);
  if (st != LPP_OK) return st;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(RW * KW * 64), p.lds, s, a);
  LPP_HIP_TRY(hipGetLastError());
  return LPP_OK;
}

// Bytes of so many partial rows: [O | max, sum].
size_t partial_bytes(size_t rows, int Dh, size_t* o_bytes) {
  if (o_bytes) *o_bytes = lpp_align_up(rows * Dh * sizeof(float), 256);
  return lpp_align_up(rows * Dh * sizeof(float), 256) + lpp_align_up(rows * 2 * sizeof(float), 256);
}
// What a call asks for, at least: room for so many ranges (bf16: all, but with less than p.share times as much none is shared; float32, which
// makes as many as there is room for: one).
size_t least_workspace(const AttnPlan& p, int ranges, int B, int H, int Dh, int L) {
  return std::min(L, kLayersPerLaunch) * partial_bytes((size_t)B * H * ranges * p.mtiles * 16, Dh, nullptr);
}
size_t partials_of(const AttnPlan& p, int B, int H, int Dh, int L, size_t* o_bytes) {
  return p.ranges < 2 ? 0 : partial_bytes((size_t)std::min(L, kLayersPerLaunch) * B * H * p.ranges * p.share * p.mtiles * 16, Dh, o_bytes);
}

}  // namespace

extern "C" size_t lpp_tree_attention_workspace(const lpp_tree* tree, int32_t B, int32_t H, int32_t S,
                                               int32_t Dh) {
  return lpp_tree_attention_layers_workspace(tree, 1, B, H, S, Dh);
}

extern "C" size_t lpp_tree_attention_layers_workspace(const lpp_tree* tree, int32_t L, int32_t B, int32_t H,
                                                      int32_t S, int32_t Dh) {
  if (!tree || L < 1 || B < 1 || H < 1 || S < 0 || (Dh != 64 && Dh != 128)) return 0;
  const AttnPlan p = plan_attention(tree, B, H, S, Dh, L);
  return std::max({least_workspace(p, p.ranges, B, H, Dh, L), partials_of(p, B, H, Dh, L, nullptr),
                   f32_workspace(tree, B, H, Dh, L, f32_splits(tree, B, H, S, L), nullptr)});
}

namespace {
int32_t tree_attention_impl(const lpp_tree* tree, int32_t dtype, int32_t out_dtype, const lpp_attention_layer* layers,
                            int32_t L, const int32_t* seq_len, int32_t B, int32_t H, int32_t Hkv, int32_t S,
                            int32_t Dh, float scale, void* ws, size_t ws_bytes, void* stream) {
  if (!tree || !layers || L < 1) return LPP_EINVAL;
  if (B < 1 || H < 1 || S < 0 || Dh < 1) return LPP_EINVAL;
  if (Hkv < 1 || Hkv > H || H % Hkv != 0) return LPP_EINVAL;
  for (int32_t l = 0; l < L; ++l) {
    const lpp_attention_layer& y = layers[l];
    if (!y.q || !y.k_tree || !y.v_tree || !y.out) return LPP_EINVAL;
    if (S > 0 && (!y.k_cache || !y.v_cache)) return LPP_EINVAL;
  }
  if (!(scale >= 0.f) || scale == INFINITY) return LPP_EINVAL;   // NaN, negative, infinite
  if (Dh != 64 && Dh != 128) return LPP_EUNSUPPORTED;
  if (dtype != LPP_F32 && dtype != LPP_BF16) return LPP_EUNSUPPORTED;
  if (out_dtype != LPP_F32 && out_dtype != LPP_BF16) return LPP_EUNSUPPORTED;
  if ((int64_t)B * H > (1 << 24) || (int64_t)B * H * H >= (1ll << 32)) return LPP_EUNSUPPORTED;
  if ((int64_t)S * Dh >= (1ll << 31) || (int64_t)tree->M * Dh >= (1ll << 31)) return LPP_EUNSUPPORTED;   // 32-bit offsets inside one head
  AttnPlan p = plan_attention(tree, B, H, S, Dh, L);
  const size_t need = least_workspace(p, dtype == LPP_F32 ? 1 : p.ranges, B, H, Dh, L);
  if (!ws || ws_bytes < need) return LPP_ENOWORKSPACE;
  if (ws_bytes < partials_of(p, B, H, Dh, L, nullptr)) p = plan_attention(tree, B, H, S, Dh, L, false);
  if (!tree->d_anc) return LPP_EHIP;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (scale == 0.f) scale = 1.0f / sqrtf((float)Dh);

  // up to kLayersPerLaunch layers per launch (bf16: fewer of more than 16384 units each); the launches of one call follow
  // each other on the stream and share the workspace
  const int64_t per_head = (int64_t)(H / Hkv) * p.msplits, padded = ((int64_t)B * Hkv + 7) / 8 * 8 * per_head;
  const int32_t most = dtype == LPP_F32 ? kLayersPerLaunch : layers_per_launch(padded, kLayersPerLaunch);
  for (int32_t l0 = 0; l0 < L; l0 += most) {
    const int32_t nl = std::min(L - l0, most);
    if (dtype == LPP_F32) {
      AttnArgsF32 a;
      for (int32_t l = 0; l < kLayersPerLaunch; ++l) {
        const lpp_attention_layer& y = layers[l0 + std::min(l, nl - 1)];
        a.layer[l] = LayerPtrs{y.q, y.k_cache, y.v_cache, y.k_tree, y.v_tree, y.out};
      }
      a.seq_len = seq_len; a.anc = tree->d_anc;
      a.B = B; a.H = H; a.Hkv = Hkv; a.S = S; a.M = tree->M; a.words = tree->words;
      a.mtiles = p.mtiles; a.gq = H / Hkv; a.out_bf16 = out_dtype == LPP_BF16;
      a.scale = scale;
      if ((int64_t)S + tree->M > kMostKeysF32) return LPP_EUNSUPPORTED;
      size_t o_bytes = 0;
      a.nsplit = f32_splits(tree, B, H, S, L);
      while (a.nsplit > 1 && f32_workspace(tree, B, H, Dh, L, a.nsplit, &o_bytes) > ws_bytes) --a.nsplit;
      const uint64_t tiles = (((uint64_t)B * Hkv + 7) / 8) * a.gq * a.mtiles * a.nsplit;
      a.rc_nsplit = reciprocal((uint32_t)a.nsplit, std::max<uint64_t>(tiles, (uint64_t)(S + tree->M) * a.nsplit));
      a.rc_per = reciprocal((uint32_t)(a.mtiles * a.gq), tiles);
      a.rc_mtiles = reciprocal((uint32_t)a.mtiles, (uint64_t)a.mtiles * a.gq);
      a.rc_Hkv = reciprocal((uint32_t)Hkv, (uint64_t)B * Hkv);
      a.ws_o = reinterpret_cast<float4*>(ws);
      a.ws_ml = reinterpret_cast<float2*>(reinterpret_cast<unsigned char*>(ws) + o_bytes);
      const int32_t st = Dh == 64 ? launch_f32<64, 16>(a, nl, s) : launch_f32<128, 8>(a, nl, s);
      if (st != LPP_OK) return st;
      continue;
    }

    AttnArgs a;
    for (int32_t l = 0; l < kLayersPerLaunch; ++l) {
      const lpp_attention_layer& y = layers[l0 + std::min(l, nl - 1)];
      a.layer[l] = LayerPtrs{y.q, y.k_cache, y.v_cache, y.k_tree, y.v_tree, y.out};
    }
    a.seq_len = seq_len; a.anc = tree->d_anc;
    a.H = H; a.S = S; a.M = tree->M; a.words = tree->words;
    a.KVBH = B * Hkv; a.gq = H / Hkv; a.out_bf16 = out_dtype == LPP_BF16;
    a.msplits = p.msplits; a.nsplit = p.ranges * p.share; a.ranges = p.ranges; a.share_bits = p.share == 2; a.rows_pad = p.mtiles * 16;
    a.scale_log2 = scale * 1.44269504088896340736f;
    // Key/value heads beyond a multiple of 8: in one layer, in few whose heads make no eight and where the keys are cut in ranges,
    // their blocks take turns on the XCDs (1 head of 4 in 4 items, 67 rows, 1313 keys 16.2 -> 9.6 us).  In more layers a head keeps to
    // an XCD, whose L2 then has its keys for all blocks that read them, and the next layer's heads to the XCDs behind (5 heads for 20,
    // 61 rows, 16 layers, 1286 keys 25 us, in turns 35).
    const bool turns = nl * (a.KVBH & 7) < 8 || nl == 1 || p.ranges > 1;        // (padding has no place among the partials)
    const int64_t upl = turns ? (int64_t)B * Hkv * per_head : padded;
    const int64_t units = upl * nl, blocks = units * a.nsplit;
    if (blocks >= (1ll << 31)) return LPP_EUNSUPPORTED;
    a.rc_msplits = reciprocal((uint32_t)p.msplits); a.rc_H = reciprocal((uint32_t)H); a.rc_nsplit = reciprocal((uint32_t)a.nsplit);
    a.rc_ranges = reciprocal((uint32_t)p.ranges);
    a.rc_gq = reciprocal((uint32_t)(H / Hkv));
    a.units_per_layer = nl == 1 ? 0xFFFFFFFFu : (uint32_t)upl;                  // (one layer: 0, however many units)
    a.rc_upl = reciprocal(a.units_per_layer);
    a.left = turns ? (uint32_t)(a.KVBH & 7) : 0u; a.rc_left = reciprocal(a.left);
    a.eights = (uint32_t)(upl - a.left * per_head);
    a.spin = turns ? 0u : (uint32_t)(a.KVBH & 7);
    a.whole_eights = (uint32_t)(units & ~7ll);
    a.units_left = (uint32_t)(units & 7); a.rc_units_left = reciprocal(a.units_left);
    // (partials only where the launch has no more blocks than compute units: they and the units are few)
    size_t o_bytes = 0;
    const size_t bytes = partials_of(p, B, H, Dh, nl, &o_bytes);
    a.counters = tree->d_counters + LPP_COUNTER_SLOTS;
    a.ws_o_bytes = (uint32_t)o_bytes; a.ws_ml_bytes = (uint32_t)(bytes - o_bytes);
    a.ws_o = reinterpret_cast<float*>(ws);
    a.ws_ml = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(ws) + o_bytes);

    int32_t st = LPP_EUNSUPPORTED;
    if (Dh == 64) {
      if (p.nt == 1) st = p.kw == 4 ? launch_bf16<64, 1, 1, 4>(a, p, blocks, s) : launch_bf16<64, 1, 1, 8>(a, p, blocks, s);
      else if (p.nt == 2) st = p.kw == 4 ? launch_bf16<64, 2, 1, 4>(a, p, blocks, s) : launch_bf16<64, 2, 1, 8>(a, p, blocks, s);
      else if (p.nt == 3) st = p.kw == 4 ? launch_bf16<64, 3, 1, 4>(a, p, blocks, s) : launch_bf16<64, 3, 1, 8>(a, p, blocks, s);
      else if (p.nt == 4) st = p.kw == 4 ? launch_bf16<64, 4, 1, 4>(a, p, blocks, s) : launch_bf16<64, 4, 1, 8>(a, p, blocks, s);
      else st = p.kw == 4 ? launch_bf16<64, 5, 1, 4>(a, p, blocks, s) : launch_bf16<64, 5, 1, 8>(a, p, blocks, s);
    } else {
      if (p.nt == 1) st = p.kw == 4 ? launch_bf16<128, 1, 1, 4>(a, p, blocks, s) : launch_bf16<128, 1, 1, 8>(a, p, blocks, s);
      else if (p.nt == 2) st = p.kw == 4 ? launch_bf16<128, 2, 1, 4>(a, p, blocks, s) : launch_bf16<128, 2, 1, 8>(a, p, blocks, s);
    }
    if (st != LPP_OK) return st;
  }
  return LPP_OK;
}
}  // namespace

extern "C" int32_t lpp_tree_attention(const lpp_tree* tree, int32_t dtype, const void* q, const void* k_cache,
                                      const void* v_cache, const void* k_tree, const void* v_tree,
                                      const int32_t* seq_len, int32_t B, int32_t H, int32_t S, int32_t Dh,
                                      float scale, float* out, void* ws, size_t ws_bytes, void* stream) {
  const lpp_attention_layer y = {q, k_cache, v_cache, k_tree, v_tree, out};
  return tree_attention_impl(tree, dtype, LPP_F32, &y, 1, seq_len, B, H, H, S, Dh, scale, ws, ws_bytes, stream);
}

extern "C" int32_t lpp_tree_attention_gqa(const lpp_tree* tree, int32_t dtype, int32_t out_dtype, const void* q,
                                          const void* k_cache, const void* v_cache, const void* k_tree,
                                          const void* v_tree, const int32_t* seq_len, int32_t B, int32_t H,
                                          int32_t Hkv, int32_t S, int32_t Dh, float scale, void* out, void* ws,
                                          size_t ws_bytes, void* stream) {
  const lpp_attention_layer y = {q, k_cache, v_cache, k_tree, v_tree, out};
  return tree_attention_impl(tree, dtype, out_dtype, &y, 1, seq_len, B, H, Hkv, S, Dh, scale, ws, ws_bytes, stream);
}

extern "C" int32_t lpp_tree_attention_layers(const lpp_tree* tree, int32_t dtype, int32_t out_dtype,
                                             const lpp_attention_layer* layers, int32_t L, const int32_t* seq_len,
                                             int32_t B, int32_t H, int32_t Hkv, int32_t S, int32_t Dh, float scale,
                                             void* ws, size_t ws_bytes, void* stream) {
  return tree_attention_impl(tree, dtype, out_dtype, layers, L, seq_len, B, H, Hkv, S, Dh, scale, ws, ws_bytes, stream);
}
