// Shared declarations of the HIP sources: storage-type helpers and the host-side launchers
// that the API file calls.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint16_t bf16_t;  // bfloat16 bit pattern

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// 16 bytes on an 8-byte boundary (a caller's bf16 tensor: what the kernels ask of it)
__device__ __forceinline__ uint4 load_16_at_8(const void* p) {
  typedef uint32_t u32x4_at_8_t __attribute__((vector_size(16), aligned(8)));
  return __builtin_bit_cast(uint4, *reinterpret_cast<const u32x4_at_8_t*>(p));
}

// round to nearest even (one v_cvt_pk_bf16_f32, which two values can share, instead of four integer operations each)
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f32_to_bf16x2(float lo, float hi) {
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
  return __builtin_bit_cast(uint32_t, (bf16x2_t){(__bf16)lo, (__bf16)hi});
}

// The attention kernels of the bf16 path take the cache in blocks of 32 positions and give what lies behind the last one a
// probability of 0, which does not cancel an infinity or NaN that an earlier, longer sequence may have left there in V.  So the
// V row is kept clear behind the last position, to the end of the 64 positions (a whole cache line: half a line costs a read of the
// other half, 29 -> 37 us on a handed-over cache of 16 x 8 x 1024) that the next one falls into: by whoever stores the last position
// of a prefill or of a handed-over cache, and by a step's append to the last of 64 positions, for the 64 behind it.  (Wide batches'
// steps mask V in their attention and clear nothing.)  next: the next position, at: its place in the row.
#define CACHE_BLOCK 64
template <typename T> __device__ __forceinline__ void clear_block(T* at, int next, int max_seq) {
  if (next >= max_seq) return;   // (the row's length is a multiple of the block's)
  int n = CACHE_BLOCK - next % CACHE_BLOCK;
  constexpr int E = 16 / sizeof(T);
  for (; n % E; --n) *at++ = T(0);
  for (; n > 0; n -= E, at += E) *reinterpret_cast<uint4*>(at) = make_uint4(0u, 0u, 0u, 0u);
}

template <typename T> __device__ __forceinline__ float load_f(const T* p);
template <> __device__ __forceinline__ float load_f<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float load_f<bf16_t>(const bf16_t* p) { return bf16_to_f32(*p); }
template <typename T> __device__ __forceinline__ void store_f(T* p, float v);
template <> __device__ __forceinline__ void store_f<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void store_f<bf16_t>(bf16_t* p, float v) { *p = f32_to_bf16(v); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// ---------------------------------------------------------------------------------------------
// launchers (host).  is_bf16 selects the storage type T of the operands marked T.
// All return the hipError_t of the launch.
// ---------------------------------------------------------------------------------------------

// x (f32 [rows][H], in place) = (emb ? emb : x_src ? x_src : x) + sum_{s<n_parts} parts[s] + sum_{j<n_peers} peers[j];
// then up to two normed copies out_a = rmsnorm(x) * gain_a, out_b likewise (T), and an optional
// f32 copy x_out.  parts: f32, slot s at parts + s*part_stride; peers: T, peer j at peers + j*peer_stride.
struct ReduceNormArgs {
  float* x;
  const void* emb;         // T [rows][H] or null
  const float* x_src;      // f32 [rows][H] or null
  const float* parts;      // f32 or null
  int n_parts;
  size_t part_stride;      // elements
  const void* peers;       // T or null
  int n_peers;
  size_t peer_stride;      // elements
  void* out_a;             // T or null
  const void* gain_a;      // T, or null = no gain
  void* out_b;
  const void* gain_b;
  float* x_out;            // f32 or null
  int x_step;              // x_out takes the step from the old rows to the new ones, not the new rows
  int rows, H;
  float eps;
};
hipError_t launch_reduce_norm(const ReduceNormArgs& a, bool is_bf16, hipStream_t s);
// a, then b on the same rows in place (bf16; no embeddings, no other source; a leaves no copy, b no step)
bool reduce_norm_two_fits(int H);
hipError_t launch_reduce_norm_two(const ReduceNormArgs& a, const ReduceNormArgs& b, hipStream_t s);

// out_a[r][:] = rmsnorm(emb[r][:]) * gain_a, out_b likewise (or null), all bf16 [rows][H], on 16-byte boundaries except emb (8); H <= 16384, a multiple of 8
#define EMBED_NORM_MAX_H 16384
hipError_t launch_embed_norm(const bf16_t* emb, bf16_t* out_a, const bf16_t* gain_a, bf16_t* out_b, const bf16_t* gain_b, int rows, int H,
                             float eps, hipStream_t s);

// The start of a pipeline stage (three tensors handed over, f32 [rows][H]; att, mlp null: zeros) in one pass: x_{-1} = res + att,
// whose normed rows are out_a, and x = x_{-1} + mlp, whose normed rows are out_b (T); x_out: an optional copy of x.  Any output of
// the stage may be one of the inputs (a thread reads its elements of all of them first).  H <= 16384.
struct StageInArgs {
  const float *res, *att, *mlp;
  float* x;
  float* x_out;            // or null
  void* out_a;
  const void* gain_a;
  void* out_b;
  const void* gain_b;
  int rows, H;
  float eps;
};
#define STAGE_IN_MAX_H 16384
hipError_t launch_stage_in(const StageInArgs& a, bool is_bf16, hipStream_t s);

// Rows of the stream as a sum that nobody has stored yet: a stored stream (emb: T, the embeddings x_0; else base: f32) and the outputs of
// the one or two modules behind it, each the partial sums of the computed shards and then the peers (order: base, parts 0.., peers 0.., ...)
struct StreamSum {
  const void* emb;
  const float* base;
  int n_adds;              // 0 .. 2
  const float* parts[2];   // f32 [n_parts][rows][H]
  int n_parts;
  size_t part_stride;      // elements
  const void* peers[2];    // T or null
  int n_peers;
  size_t peer_stride;      // elements
};
// x_out[r][:] = the sum, f32
hipError_t launch_stream_sum(const StreamSum& a, float* x_out, int rows, int H, bool is_bf16, hipStream_t s);

// Plain projections of the rows x (T [shard][M][K]) for all computed shards at once; w: T [K][N], a shard's matrices
// w_stride BYTES behind the previous shard's, as are its caches (cache_stride); the other strides are elements per shard.
enum { PLAIN_OUT = 0, PLAIN_SWIGLU = 1, PLAIN_QKV = 2 };
struct PlainGemmArgs {
  const void* x;
  size_t x_stride;         // 0: every shard reads the same rows
  int M, K, n_shards;
  int n_mat;               // matrices: 1 (OUT), gate and up (SWIGLU, equal N), q, k and v (QKV)
  const void* w[3];
  int N[3];
  size_t w_stride;
  int epilogue;
  float* out;              // OUT: f32 [shard][M][N]
  size_t out_stride;
  void* act;               // SWIGLU: T [shard][M][N] = silu(gate) * up
  size_t act_stride;
  // QKV: row b*T + t is token t of sequence b at position pos0 + t; q rotated -> T [shard][M][nq*d], k rotated and v -> the
  // caches (layouts as below)
  void* q_out;
  size_t q_stride;
  void* cache_k;
  void* cache_v;
  size_t cache_stride;
  const float* cos_tab;    // [max_seq][d/2]
  const float* sin_tab;
  int T, pos0, nkv, d, max_seq;
  // gain non-null (QKV and SWIGLU, M <= PLAIN_NORM_ROWS): instead of x the rows are rmsnorm(in) * gain, made where they are multiplied, and
  // the new rows of the stream are left in x_store (f32 [M][K], or null; not what `in` reads)
  const void* gain;
  StreamSum in;
  float eps;
  float* x_store;
  int held;                // workgroups that may count on a place of two per CU: PLAIN_HELD_WORKGROUPS, or 0
  int n_blocks;            // set by the launcher: column blocks of all matrices
};
#define PLAIN_NORM_ROWS 64
#define PLAIN_HELD_WORKGROUPS 512   // two on each of 256 CUs
// a plain matrix of N columns is read four weights at a time
inline bool plain_four_at_once(const void* w, int N) { return N % 4 == 0 && ((uintptr_t)w & 15) == 0; }
// workgroups of a plain projection of at most PLAIN_NORM_ROWS rows: 64 columns, and four rows where there is more than one
inline long long plain_workgroups(int rows, int col_blocks, int n_shards) { return (long long)(rows == 1 ? 1 : (rows + 3) / 4) * col_blocks * n_shards; }
hipError_t launch_plain_gemm(const PlainGemmArgs& a, bool is_bf16, hipStream_t s);

// qkv: f32 [n_parts][rows][(nq+2nkv)*d] (slots summed).  rows = B*T, row = b*T + t, position = pos0 + t.
// q -> T [rows][nq*d] rotated; k rotated -> cache_k T [B_cap][nkv][max_seq][d]; v -> cache_v kept
// TRANSPOSED, T [B_cap][nkv][d][max_seq] (positions contiguous: the layout the P*V contraction wants).
// max_seq here is the cache row capacity (a multiple of 64).
struct RopeAppendArgs {
  const float* qkv;
  int n_parts;
  size_t part_stride;
  void* q_out;
  void* cache_k;
  void* cache_v;
  const float* cos_tab;    // [max_seq][d/2]
  const float* sin_tab;
  int B, T, pos0, nq, nkv, d, max_seq;
  const int* pos_dev;      // if non-null the position is read from device memory (pos0 ignored)
};
hipError_t launch_rope_append(const RopeAppendArgs& a, hipStream_t s);   // T = bf16

// plain causal GQA attention over the cache, all computed shards
struct AttnGenericArgs {
  const void* q;           // T [shard][rows][nq*d]
  const void* cache_k;     // T [B_cap][nkv][max_seq][d]
  const void* cache_v;     // T [B_cap][nkv][d][max_seq]
  void* o;                 // T [shard][rows][nq*d]
  int B, T, pos0, nq, nkv, d, max_seq, n_shards;
  size_t q_stride;         // elements, of q and o
  size_t cache_stride;     // bytes
};
hipError_t launch_attn_generic(const AttnGenericArgs& a, bool is_bf16, hipStream_t s);
// A layer of at most PLAIN_NORM_ROWS rows whose modules do not read each other's output, in three launches: { qkv, gate_up }, { attn, down }, and the
// attention's output projection; whether the rule takes it
bool plain_beside(const PlainGemmArgs& qkv, const AttnGenericArgs& attn, const PlainGemmArgs& gate_up, const PlainGemmArgs& down, bool is_bf16);
hipError_t launch_plain_inputs(PlainGemmArgs a, PlainGemmArgs b, bool is_bf16, hipStream_t s);
hipError_t launch_plain_attn_beside(const AttnGenericArgs& a, PlainGemmArgs b, bool is_bf16, hipStream_t s);
// ... or in two for a single row, { qkv, gate_up }, { attn + its output projection, down }, where plain_attn_out_fits
#define PLAIN_ATTN_OUT_POSITIONS 256   // times heads: a chunk of 64 for each of four wavefronts
bool plain_attn_out_fits(const AttnGenericArgs& a, const PlainGemmArgs& o, const PlainGemmArgs& down, bool is_bf16);
hipError_t launch_plain_attn_out(const AttnGenericArgs& a, PlainGemmArgs o, PlainGemmArgs b, bool is_bf16, hipStream_t s);

// act[m][i] = silu(gate) * up from the partial products of the packed gate/up projection (tile columns 0..7 gate, 8..15 the matching up
// columns), act bf16: parts f32 [n_parts][M][2I], slot s at parts + s * part_stride, summed in slot order
struct SwigluPartsArgs {
  const float* parts;
  int n_parts;
  size_t part_stride;      // elements
  bf16_t* act;
  int M, I;
};
hipError_t launch_swiglu_parts(const SwigluPartsArgs& a, hipStream_t s);
hipError_t launch_rope_swiglu(const RopeAppendArgs& a, const SwigluPartsArgs& b, hipStream_t s);   // both in one launch

// ---- generation head ----------------------------------------------------------------------------
// x_out[r][:] = table[tokens[r]][:]  (T [rows][H]); an id outside [0, vocab) reads the nearest valid row and sets
// *bad_id (host-visible memory, may be null) to 1
hipError_t launch_embed_gather(const int* tokens, const void* table, void* x_out, int rows, int H, int vocab,
                               unsigned* bad_id, bool is_bf16, hipStream_t s);
// y[r][:] = x[r][:] / sqrt(mean(x[r]^2) + eps) * gain   (gain may be null = 1); y: T [rows][H], or (tiled, H % 8 == 0) [H / 8][rows][8]
hipError_t launch_head_norm(const float* x, const void* gain, void* y, int rows, int H, float eps, bool tiled, bool is_bf16,
                            hipStream_t s);
// tokens_out[r] = index of the largest of logits[r][0..V), the lowest index among equal maxima
// (scratch: memory of scratch_per_row bytes per row that nothing needs any more; may be null with 0)
hipError_t launch_argmax(const float* logits, int* tokens_out, int rows, int V, void* scratch, size_t scratch_per_row, hipStream_t s);

// ---- bf16 streaming / MFMA path ----------------------------------------------------------------
// Packed weight format ("tiles"): the [K][N] matrix is cut into tiles of 32 k x 16 n; tile (nt, kt)
// is 1 KiB at ((nt*KT + kt)*64 + lane)*16 bytes, lane holding W[kt*32 + (lane/16)*8 + e][nt*16 + lane%16]
// for e = 0..7 -- exactly one wavefront's A operand of a 16x16x32 bf16 MFMA, so a wave reads a tile
// with one fully coalesced 16-byte-per-lane load.  K and N are zero-padded to multiples of 32 / 16.
static inline size_t packed_tiles_bytes(int K, int N) {
  return (size_t)((N + 15) / 16) * (size_t)((K + 31) / 32) * 1024;
}
// Repack src (bf16 [K][N], row stride N) into dst tiles at column-tile offset: column n of src becomes
// packed column map(n).  mode 0: n -> col0 + n.  mode 1 (gate) / 2 (up): SwiGLU interleave,
// n -> 16*(n/8) + (n%8) + (mode==2 ? 8 : 0), so each 16-wide tile holds 8 gate and the 8 matching up columns.
// The values are copied bit for bit.
hipError_t launch_repack_tiles(const bf16_t* src, void* dst, int K, int N, int N_total, int col0, int mode, hipStream_t s);

struct GemvArgs {
  const bf16_t* x;         // bf16 [M][ldx], or (x_tiled) [K / 8][M][8]: what a wavefront reads of a k tile is one piece of memory
  int ldx;
  int x_tiled;
  const void* wp;          // packed tiles, N_total columns, K rows
  int M, K, N;             // N = packed column count (multiple of 16 after padding)
  int ksplit;              // workgroups along K; out slot = slot0 + ks
  float* out;              // epilogue 0: f32 [slot][M][N] partial sums, slot stride out_stride
  size_t out_stride;
  int slot0;
  bf16_t* act;             // epilogue 1 (ksplit must be 1): SwiGLU -> bf16 [M][N/2]
  int epilogue;
};
// launch shape of the skinny GEMM for a problem: column tiles per workgroup, wavefronts per workgroup,
// k tiles per register buffer, workgroups along K (1 unless allow_ksplit)
struct GemvPlan { int tn, waves, u, ksplit; };
GemvPlan gemv_plan(int N, int K, bool allow_ksplit);
hipError_t launch_gemv(const GemvArgs& a, hipStream_t s);

struct AttnDecodeArgs {
  const bf16_t* q;         // [B][nq*d] rotated
  const bf16_t* cache_k;   // [B_cap][nkv][max_seq][d]
  const bf16_t* cache_v;   // [B_cap][nkv][d][max_seq]
  float* part_o;           // [B][nkv][n_splits][g][d]
  float* part_ml;          // [B][nkv][n_splits][g][2]
  bf16_t* o;               // [B][nq*d]
  int B, nq, nkv, d, max_seq;
  int n_pos;               // visible positions (incl. the new one)
  int n_splits;            // workgroups per (sequence, kv head); attn_decode_splits()
  const int* pos_dev;      // if non-null: n_pos = *pos_dev + 1
};
#define ATTN_DECODE_MAX_SPLITS 512
int attn_decode_splits(int B, int nkv, int max_seq);   // (the grid depends on the capacity, not on the position)
hipError_t launch_attn_decode(const AttnDecodeArgs& a, hipStream_t s);

// ---- prefill MFMA path ---------------------------------------------------------------------------
struct GemmArgs {
  const bf16_t* x;         // bf16 [M][ldx]
  int ldx;
  const void* wp;          // packed tiles
  int M, K, N;
  float* out;              // epilogue 0: f32 [M][N] (row stride N)
  bf16_t* act;             // epilogue 1: SwiGLU -> bf16 [M][N/2]
  int epilogue;
  // epilogue 2: the columns are q | k | v heads of d columns each; row m is token m % T of sequence m / T at
  // position pos0 + m % T: rotary embedding of q and k (adjacent pairs), q -> q_out bf16 [M][nq*d], k and v ->
  // the cache (k [seq][nkv][max_seq][d], v transposed [seq][nkv][d][max_seq])
  bf16_t* q_out;
  bf16_t* cache_k;
  bf16_t* cache_v;
  const float* cos_tab;    // [max_seq][d/2]
  const float* sin_tab;
  int T, pos0, nq, nkv, d, max_seq;
  // epilogue 3: the residual update of Algorithm 1 (a module's reduced output joins the stream) with the AllReduce written as a sum
  // over rank partial sums (Eq. 2): x_res[m][n] = x_res[m][n] + product + peers_0[m][n] + peers_1[m][n] + ...
  // (in this order, in place, row stride N), an optional f32 copy, for each module that reads the new rows a bf16
  // copy of them times the gain of that module's RMSNorm (the product in fp32, one rounding), and the rows' sums
  // of squares per column block: ssq_part[block][m], gemm_ssq_parts() blocks
  float* x_res;
  const bf16_t* x_emb;     // if non-null the old rows are these (the embeddings, bf16 [M][N]) and not what x_res holds
  int last;                // the new rows are not left in x_res: nothing reads the stream after this module
  float* x_copy;           // or null
  int copy_step;           // the copy is the step from the old rows to the new ones (a module output that a stage hands over), not the new rows
  bf16_t* xh_a;            // bf16 [M][N], or null
  const bf16_t* gain_a;    // bf16 [N] (with xh_a)
  bf16_t* xh_b;            // or null (only with xh_a)
  const bf16_t* gain_b;    // bf16 [N] (with xh_b)
  const bf16_t* peers;     // bf16 [n_peers][peer_stride], row stride N; or null
  int n_peers;
  size_t peer_stride;      // elements
  float* ssq_part;         // f32 [gemm_ssq_parts()][M] (at most ceil(N / 32) blocks), or null
  // every epilogue: if non-null, row m of the product is multiplied by row_scale[m] first (the 1/rms of an
  // RMSNorm whose gain the producer of x has already applied: the factor commutes with the product)
  const float* row_scale;
  // epilogue 0 only: workgroups along K; split ks leaves its partial product in out + ks * out_stride (0 or 1: no split)
  int ksplit;
  size_t out_stride;       // elements
};
hipError_t launch_gemm_mfma(const GemmArgs& a, hipStream_t s);
// two products that do not depend on each other in one launch, where there is a kernel for their tiles (gemm_pairs)
bool gemm_pairs(const GemmArgs& a, const GemmArgs& b);
hipError_t launch_gemm_pair(const GemmArgs& a, const GemmArgs& b, hipStream_t s);
// epilogue 0: the number of workgroups along K (1 .. max_split) that suits an M x N x K product
// (extra_us: what taking a split at all costs beside the product)
int gemm_ksplit(int M, int N, int K, int max_split, float extra_us);
int gemm_ssq_parts(const GemmArgs& a);   // epilogue 3: the number of column blocks that launch_gemm_mfma(a) leaves in ssq_part
// rs_a[m] (and rs_b[m] if non-null) = 1 / sqrt(sum_p ssq_part[p][m] / H + eps), p < n_part, fixed summation order
hipError_t launch_row_rms(const float* ssq_part, int n_part, int M, int H, float eps, float* rs_a, float* rs_b, hipStream_t s);

struct AttnPrefillArgs {
  const bf16_t* q;         // [B*T][nq*d] rotated
  const bf16_t* cache_k;   // [B_cap][nkv][max_seq][d]
  const bf16_t* cache_v;   // [B_cap][nkv][d][max_seq]
  bf16_t* o;               // [B*T][nq*d]
  int B, T, pos0, nq, nkv, d, max_seq;
};
hipError_t launch_attn_prefill(const AttnPrefillArgs& a, hipStream_t s);

// transposes caller-made V content [B][nkv][S][d] into the cache layout [B_cap][nkv][d][max_seq] and copies K (clear: see clear_block)
hipError_t launch_load_kv(const void* k, const void* v, void* cache_k, void* cache_v, int B, int nkv, int S, int d,
                          int max_seq, bool is_bf16, bool clear, hipStream_t s);
