// Internal launchers behind the C ABI (host side).  Arguments are validated
// by the ABI layer before any of these is called.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace sfa {

hipError_t launch_topk_encode(const float* x, int64_t rows, int d, int k, void* idx, int ifmt,
                              void* val, int vfmt, hipStream_t stream);

hipError_t launch_attn_fwd(const void* q_idx, const void* q_val, const void* k_idx,
                           const void* k_val, const void* v, int B, int Hq, int Hkv, int n, int d,
                           int k, int causal, int window, int n_global, float scale, int ifmt,
                           int vfmt, int vbf16, int obf16, void* o, float* lse, void* ws,
                           hipStream_t stream);
int fwd_max_group();
size_t fwd_workspace_bytes(int B, int Hkv, int n, int d, int vbf16);

// forward at float32 accuracy for head dimensions (d <= 256) and group sizes
// without the tuned kernel; no workspace
hipError_t launch_attn_fwd_generic(const void* q_idx, const void* q_val, const void* k_idx,
                                   const void* k_val, const void* v, int B, int Hq, int Hkv,
                                   int n, int d, int k, int causal, int window, int n_global,
                                   float scale, int ifmt, int vfmt, int vbf16, int obf16, void* o,
                                   float* lse, hipStream_t stream);
bool fwd_generic_supported(int d, int k);

hipError_t launch_attn_bwd(const void* q_idx, const void* q_val, const void* k_idx,
                           const void* k_val, const void* v, const void* o, const float* lse,
                           const void* dout, int B, int Hq, int Hkv, int n, int d, int k,
                           int causal, int window, int n_global, float scale, int ifmt,
                           int vfmt, int vbf16, int obf16, float* dq, float* dk, float* dv,
                           void* ws, hipStream_t stream);
size_t bwd_workspace_bytes(int B, int Hq, int Hkv, int n, int d);
int bwd_max_group();

// float32 backward for head dimensions without the matrix-core kernels
// (d <= 256); no workspace, any group size
hipError_t launch_attn_bwd_generic(const void* q_idx, const void* q_val, const void* k_idx,
                                   const void* k_val, const void* v, const void* o,
                                   const float* lse, const void* dout, int B, int Hq, int Hkv,
                                   int n, int d, int k, int causal, int window, int n_global,
                                   float scale, int ifmt, int vfmt, int vbf16, int obf16,
                                   float* dq, float* dk, float* dv, hipStream_t stream);
bool bwd_generic_supported(int d, int k);

hipError_t launch_attn_fwd_index(const void* q_idx, const void* q_val, const void* k_idx,
                                 const void* k_val, const void* v, int B, int Hq, int Hkv, int n,
                                 int d, int k, int causal, float scale, int ifmt, int vfmt,
                                 int vbf16, int obf16, void* o, float* lse, hipStream_t stream);
int fwd_index_lds_bytes(int d, int k, int vbf16);
int fwd_index_max_k();
int fwd_index_rows_per_block();

// Decode over a contiguous (table == nullptr: [B, Hkv, Lmax, ...]) or paged
// (pages [num_pages, Hkv, 1 << log2P, ...], table [B, max_pages],
// Lmax = max_pages << log2P) cache; query codes, or q_dense coded in-kernel.
struct DecodeArgs {
  const float* q_dense;
  const void *q_idx, *q_val, *kc_idx, *kc_val, *v;
  const int32_t* seq_len;
  const int32_t* table;
  int B, Hq, Hkv, Lmax, d, k;
  int max_pages, log2P, num_pages;
  int window, n_global;  // token pattern (window 0: none)
  float scale;
  int qifmt, qvfmt, kifmt, kvfmt, vbf16, obf16;
  void* o;
  float* lse;
  void* ws;
  int aim;  // tuned decode: decode_chunks_aim, or 0 where ws holds kDecodeChunk chunks only
  // 8-bit cache (launch_attn_decode_q8): float32 scale per key row / value row
  const float* kc_scale;
  const float* v_scale;
};
// Most keys of a decode workgroup (one context chunk), and of the float32
// decode's; the workspace holds one partial (m, l, o) per chunk, query head
// and sequence.
constexpr int kDecodeChunk = 4096;
// Fewest keys of a chunk (64 per wavefront), and the workgroups that the
// tuned decode aims at by cutting sequences into smaller chunks (decode_plan):
// one per compute unit; more for the 8-bit cache, whose waves do more
// arithmetic per byte, and under a token window, which fills its first and
// last chunk only partly.
constexpr int kDecodeMinChunk = 256;
constexpr int kDecodeTarget = 256, kDecodeTargetQ8 = 1024, kDecodeTargetWindow = 2048;
// Chunks per (sequence, KV head) that a step over B * Hkv of them aims at.
// 0: every chunk has kDecodeChunk keys (B * Hkv alone passes the target); 1: the same,
// but a sequence that fits one smaller chunk has that.
inline int decode_chunks_aim(int B, int Hkv, bool q8, int window) {
  const int target = window > 0 ? kDecodeTargetWindow : q8 ? kDecodeTargetQ8 : kDecodeTarget;
  return (int)(target / ((int64_t)B * Hkv));
}
// Partial slots per (sequence, query head) of a step that reads at most
// `span` keys of each sequence with that aim (decode_plan).
inline int decode_slots(int span, int aim) {
  auto up = [](int a, int b) { return a / b + (a % b != 0); };
  const int big = up(span, kDecodeChunk), fine = up(span, kDecodeMinChunk);
  const int most = aim > big ? aim : big;
  return fine < most ? fine : most;
}
hipError_t launch_attn_decode(const DecodeArgs& a, hipStream_t stream);
// Workspace of any step of these sizes, and of one in chunks of kDecodeChunk
// keys (never more than the former).
size_t decode_workspace_bytes(int B, int Hq, int Lmax, int d);
size_t decode_workspace_bytes_min(int B, int Hq, int Lmax, int d);
// The aim of a step with a workspace of ws_bytes (at least the minimum).
int decode_aim(int B, int Hq, int Hkv, int Lmax, int d, int window, size_t ws_bytes, bool q8);
int decode_max_group();
// float32 decode for head dimensions without the tuned kernel (d <= 256);
// same partial layout, in chunks of kDecodeChunk keys; Hq / Hkv <= decode_max_group()
hipError_t launch_attn_decode_generic(const DecodeArgs& a, hipStream_t stream);

// Static device scratch of the allocation-free decode (one copy per GPU):
// its size, and its device address on the current device (looked up once per
// device).
size_t noalloc_scratch_bytes();
hipError_t noalloc_scratch(void** out);

// Decode over the 8-bit cache: int8 code values (int16 indices, k in
// {8, 16, 32}) and int8 value rows with their scales; d in {64, 128}, Hq /
// Hkv a power of two <= 8.
hipError_t launch_attn_decode_q8(const DecodeArgs& a, hipStream_t stream);
bool decode_q8_supported(int d, int k, int G);

// KV-cache append: Top-k coding of new keys and copy of their values into a
// contiguous (table == nullptr: [B, Hkv, P, ...]) or paged cache, then
// seq_len[b] += the appended count (clamped to the capacity).
struct AppendArgs {
  const float* k_new;
  const void* v_new;
  const int32_t* n_new;
  int32_t* seq_len;
  const int32_t* table;
  void *kc_idx, *kc_val, *v_cache;
  int B, Hkv, T, d, k;
  int page_size, max_pages, num_pages;
  int log2P;  // paged: page_size == 1 << log2P
  int ifmt, vfmt, vin_bf16, vc_bf16;
  // 8-bit cache: kc_val and v_cache hold int8, with one float32 scale per
  // key row (kc_scale) and value row (v_scale)
  int q8;
  float* kc_scale;
  float* v_scale;
};
hipError_t launch_kv_append(const AppendArgs& a, hipStream_t stream);

// CSR codes (row r: entries indptr[r] .. indptr[r+1]-1) to fixed rows of kmax
// entries, padded with zero values at the lowest free coordinates.
struct CsrArgs {
  const int32_t* indptr;
  const void* indices;
  const void* values;
  int64_t rows;
  int d, kmax;
  int ifmt_in, vbytes;  // index format; value storage bytes (copied bitwise)
  void* idx_out;
  int ifmt_out;
  void* val_out;
};
hipError_t launch_csr_to_codes(const CsrArgs& a, hipStream_t stream);

}  // namespace sfa
