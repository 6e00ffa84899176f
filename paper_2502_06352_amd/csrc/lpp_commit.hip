// Commit of a verified step to the KV cache (paper App. A.2 "Tree drafting and decoding":
// accepted tokens are kept, what follows the first rejection is discarded): the K/V rows of the
// root and of the accepted path are appended to each item's cache in path order.
//
// Pure data movement, at most (1 + depth) rows of Dh elements per (batch, head): one block per
// (batch*head, slot), 16 bytes per lane.  Bound by the loads that wait for each other: the arguments, then the accepted
// length, the item's length and the path entry side by side (one after the other, and the rows of V behind those of K, a step of four items took 0.6 us more),
// then the rows.
#include "lpp_internal.h"

namespace {

struct CommitArgs {
  const unsigned char* kt;
  const unsigned char* vt;
  unsigned char* kc;
  unsigned char* vc;
  const int32_t* path;
  const int32_t* accept_len;
  const int32_t* seq_len;
  int32_t* new_len;
  int32_t H, S, M, depth;
  int32_t row_bytes;      // Dh * element size
  uint32_t rc_H;          // ceil(2^32 / H): block / H as the upper half of a product (exact while blocks * H < 2^32); 0: H = 1; 1: divide
};

__global__ __launch_bounds__(64) void commit_kv_kernel(CommitArgs a) {
  const int bh = blockIdx.x, slot = blockIdx.y;          // slot 0 = root, slot i = path[i - 1]
  int H = a.H;
  uint32_t rc_H = a.rc_H;
  asm("" : "+s"(H), "+s"(rc_H) : "s"(a.kt), "s"(a.vt), "s"(a.kc), "s"(a.vc), "s"(a.path), "s"(a.accept_len), "s"(a.seq_len), "s"(a.new_len),
      "s"(a.S), "s"(a.M), "s"(a.depth), "s"(a.row_bytes));
  const int b = rc_H <= 1 ? (int)(rc_H == 0 ? (uint32_t)bh : (uint32_t)bh / (uint32_t)H) : (int)(((uint64_t)(uint32_t)bh * rc_H) >> 32);
  int accepted = a.accept_len[b], len = a.seq_len[b], node = a.path[(int64_t)b * a.depth + max(slot - 1, 0)];
  asm("" : "+s"(accepted), "+s"(len), "+s"(node));
  const int n = min(max(accepted, 0), a.depth);
  const int base = min(max(len, 0), a.S);
  if (slot == 0 && bh == b * H && threadIdx.x == 0 && a.new_len) a.new_len[b] = min(base + 1 + n, a.S);
  if (slot > n) return;
  const int pos = base + slot;
  if (pos >= a.S) return;                                  // past the capacity: dropped
  const int row = slot > 0 ? min(max(node, 0), a.M - 1) : 0;     // (M = 1: the root, whatever was read)
  const int64_t src = ((int64_t)bh * a.M + row) * a.row_bytes, dst = ((int64_t)bh * a.S + pos) * a.row_bytes;
  for (int o = threadIdx.x * 16; o < a.row_bytes; o += 64 * 16) {
    const uint4 k = *reinterpret_cast<const uint4*>(a.kt + src + o), v = *reinterpret_cast<const uint4*>(a.vt + src + o);
    *reinterpret_cast<uint4*>(a.kc + dst + o) = k;
    *reinterpret_cast<uint4*>(a.vc + dst + o) = v;
  }
}

}  // namespace

extern "C" int32_t lpp_commit_kv(const lpp_tree* tree, int32_t dtype, const void* k_tree, const void* v_tree,
                                 const int32_t* path, const int32_t* accept_len, const int32_t* seq_len,
                                 int32_t B, int32_t H, int32_t S, int32_t Dh, void* k_cache, void* v_cache,
                                 int32_t* new_len, void* stream) {
  if (!tree || !k_tree || !v_tree || !path || !accept_len || !seq_len || !k_cache || !v_cache) return LPP_EINVAL;
  if (B < 1 || H < 1 || S < 1 || Dh < 1) return LPP_EINVAL;
  if (new_len == seq_len) return LPP_EINVAL;                // every head's block reads seq_len
  if (dtype != LPP_F32 && dtype != LPP_BF16) return LPP_EUNSUPPORTED;
  const int esz = dtype == LPP_F32 ? 4 : 2;
  if ((Dh * esz) % 16 != 0) return LPP_EUNSUPPORTED;
  if ((int64_t)B * H > 0x7FFFFFFF) return LPP_EUNSUPPORTED;
  if (!tree->d_anc) return LPP_EHIP;                         // host-only handle: no device
  CommitArgs a;
  a.kt = (const unsigned char*)k_tree; a.vt = (const unsigned char*)v_tree;
  a.kc = (unsigned char*)k_cache; a.vc = (unsigned char*)v_cache;
  // (a tree of the root alone has no path entries, [B, 0]: what the kernel reads ahead is then something else of B words)
  a.path = tree->depth > 0 ? path : seq_len; a.accept_len = accept_len; a.seq_len = seq_len; a.new_len = new_len;
  a.rc_H = H == 1 ? 0u : ((int64_t)B * H * H < (1ll << 32) ? (uint32_t)(((1ll << 32) + H - 1) / H) : 1u);
  a.H = H; a.S = S; a.M = tree->M; a.depth = tree->depth > 0 ? tree->depth : 1;
  a.row_bytes = Dh * esz;
  hipLaunchKernelGGL(commit_kv_kernel, dim3((unsigned)(B * H), (unsigned)(a.depth + 1)), dim3(64), 0,
                     reinterpret_cast<hipStream_t>(stream), a);
  LPP_HIP_TRY(hipGetLastError());
  return LPP_OK;
}
