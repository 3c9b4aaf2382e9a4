// Decode-shape kernels of the bf16 path (gfx950): weight repacking into MFMA tiles, the
// weight-streaming skinny GEMM, and split-KV attention over the cache with its combine step.
#include "common.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

// ------------------------------------------------------------------------------------------------
// Repack: one thread per (tile, lane); writes the lane's 8 consecutive k of its packed column.
// ------------------------------------------------------------------------------------------------
__global__ void repack_tiles_kernel(const bf16_t* __restrict__ src, uint4* __restrict__ dst, int K, int N,
                                    int N_total, int col0, int mode) {
  const int KT = (K + 31) / 32, NT = (N_total + 15) / 16;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)NT * KT * 64) return;
  const int lane = (int)(gid & 63);
  const long long tile = gid >> 6;
  const int kt = (int)(tile % KT), nt = (int)(tile / KT);
  const int pc = nt * 16 + (lane & 15);
  int n_src;
  if (mode == 0) {
    n_src = pc - col0;
  } else {
    const int in_tile = pc & 15;
    if ((mode == 1) != (in_tile < 8)) return;  // gate owns the low 8 columns of a tile, up the high 8
    n_src = 8 * (pc >> 4) + (in_tile & 7);
  }
  if (n_src < 0 || n_src >= N) return;
  const int k0 = kt * 32 + (lane >> 4) * 8;
  uint32_t w[4];
  for (int e = 0; e < 4; ++e) {
    const int ka = k0 + 2 * e, kb = ka + 1;
    const uint32_t lo = ka < K ? src[(size_t)ka * N + n_src] : 0;
    const uint32_t hi = kb < K ? src[(size_t)kb * N + n_src] : 0;
    w[e] = lo | (hi << 16);
  }
  dst[gid] = make_uint4(w[0], w[1], w[2], w[3]);
}

hipError_t launch_repack_tiles(const bf16_t* src, void* dst, int K, int N, int N_total, int col0, int mode, hipStream_t s) {
  const long long total = (long long)((N_total + 15) / 16) * ((K + 31) / 32) * 64;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  hipLaunchKernelGGL(repack_tiles_kernel, dim3(blocks), dim3(256), 0, s, src, (uint4*)dst, K, N, N_total, col0, mode);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Weight-streaming skinny GEMM  out[m][n] = sum_k x[m][k] W[k][n]  for M <= 16 rows
// (more rows: gemm_ring_kernel, prefill_kernels.hip).
// HBM-bound: every weight byte is read once, as one coalesced 1 KiB tile per wavefront load
// (non-temporal: the stream must not evict x from the caches), and goes straight into the A operand
// of a 16x16x32 bf16 MFMA; the B operand is the matching 16 rows x 32 k slice of x (rows >= M zeroed),
// read from L1/L2 once per k tile and shared by the wave's TN column tiles (where the producer can lay it out so, x_tiled, as
// one piece of memory instead of 64 bytes from each row: head of 128256 logits, hidden 4096, 16 rows 199 -> 185 us, 4096 x 32000 59.8 -> 54.9; four
// rows and fewer no different.  Four column tiles instead, which read it half as often: 16 rows 199 / 204, one row 168 / 189).  A workgroup owns TN
// adjacent 16-column tiles and a K range; its WAVES wavefronts split that range and add up through
// LDS in a fixed order (wave 0.., then the ksplit slots by the consumer).
// Latency hiding is explicit: two register buffers of U k-tiles each, the next batch is always in
// flight while the current one is multiplied.  All loads are unconditional (addresses clamped into
// the wave's range, contributions masked at use) and the K loop is wave-uniform, so the compiler can
// count outstanding loads exactly instead of draining them.
// ------------------------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;

template <int WAVES, int U, int TN>
__global__ __launch_bounds__(WAVES * 64) void gemv_mfma_kernel(GemvArgs a) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int b = lane & 15, q = lane >> 4;
  const int nt0 = blockIdx.x * TN, ks = blockIdx.y;
  const int KT = a.K >> 5;
  const int kt_per_wg = (KT + a.ksplit - 1) / a.ksplit;
  const int wg0 = ks * kt_per_wg;
  const int wg1 = min(KT, wg0 + kt_per_wg);
  // the wavefronts take groups of U k tiles round robin: the workgroup sweeps its weight range once (DRAM page
  // locality: measured faster than a contiguous share per wavefront)
  constexpr int KB = WAVES * U, KA = 2 * WAVES * U;   // tile distance to the second register buffer / to the next turn
  const int kt0 = wg0 + wave * U;
  const int kt1 = wg1;

  f32x4_t acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) acc[j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

  const u32x4_t* wptr = reinterpret_cast<const u32x4_t*>(a.wp) + ((size_t)nt0 * KT) * 64 + lane;
  const bool rowok = b < a.M;
  const int x_kt = a.x_tiled ? 32 * a.M : 32;   // elements per k tile
  const bf16_t* xptr = a.x + (a.x_tiled ? (size_t)(q * a.M + min(b, a.M - 1)) * 8 : (size_t)min(b, a.M - 1) * a.ldx + q * 8);
  u32x4_t wa[TN][U], wb[TN][U], xa[U], xb[U];
  auto load = [&](u32x4_t (&wv)[TN][U], u32x4_t (&xv)[U], int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ktc = min(kt + u, kt1 - 1);
#pragma unroll
      for (int j = 0; j < TN; ++j) wv[j][u] = __builtin_nontemporal_load(wptr + ((size_t)j * KT + ktc) * 64);
      xv[u] = *reinterpret_cast<const u32x4_t*>(xptr + (size_t)ktc * x_kt);
    }
  };
  auto fma = [&](const u32x4_t (&wv)[TN][U], const u32x4_t (&xv)[U], int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool kok = kt + u < kt1;
      const u32x4_t xz = (kok && rowok) ? xv[u] : (u32x4_t){0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wv[j][u]),
                                                        __builtin_bit_cast(bf16x8_t, xz), acc[j], 0, 0, 0);
    }
  };
  if (kt0 < kt1) {
    load(wa, xa, kt0);
    for (int kt = kt0; kt < kt1; kt += KA) {
      load(wb, xb, kt + KB);
      __builtin_amdgcn_sched_barrier(0);
      fma(wa, xa, kt);
      __builtin_amdgcn_sched_barrier(0);
      load(wa, xa, kt + KA);
      __builtin_amdgcn_sched_barrier(0);
      fma(wb, xb, kt + KB);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // acc[j][r] = out[row = b][col = (nt0 + j)*16 + 4q + r]; reduce over the waves through LDS
  __shared__ float red[WAVES][TN][16][17];  // [wave][tile][col in tile][row]
  const int I = a.N >> 1;
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][j][4 * q + r][b] = acc[j][r];
  __syncthreads();
  if (a.epilogue == 0) {
    for (int i = threadIdx.x; i < TN * 256; i += WAVES * 64) {
      const int j = i >> 8, row = (i >> 4) & 15, col16 = i & 15;
      const int col = (nt0 + j) * 16 + col16;
      if (row < a.M && col < a.N) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) v += red[w][j][col16][row];
        a.out[(size_t)(a.slot0 + ks) * a.out_stride + (size_t)row * a.N + col] = v;
      }
    }
  } else {
    // SwiGLU: tile columns 0..7 are gate columns 8nt..8nt+7, columns 8..15 the matching up columns
    for (int i = threadIdx.x; i < TN * 128; i += WAVES * 64) {
      const int j = i >> 7, row = (i >> 3) & 15, c8 = i & 7;
      const int col = (nt0 + j) * 8 + c8;
      if (row < a.M && col < I) {
        float g = 0.f, u = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
          g += red[w][j][c8][row];
          u += red[w][j][c8 + 8][row];
        }
        a.act[(size_t)row * I + col] = f32_to_bf16(g / (1.0f + __expf(-g)) * u);
      }
    }
  }
}

GemvPlan gemv_plan(int N, int K, bool allow_ksplit) {
  GemvPlan p;
  const int NT = N / 16, KT = K / 32;
  p.tn = (NT <= 192 && NT % 4 == 0) ? 4 : 2;
  p.waves = KT >= 64 ? 8 : 4;
  const int groups = NT / p.tn;
  p.ksplit = 1;
  if (allow_ksplit)
    while (groups * p.ksplit * p.waves < 1536 && KT / (p.ksplit * 2 * p.waves) >= 8 && p.ksplit < 8) p.ksplit *= 2;
  p.u = p.waves == 4 && p.tn == 2 ? 4 : 2;
  return p;
}

hipError_t launch_gemv(const GemvArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.M > 16 || (a.N & 31) || (a.K & 31)) return hipErrorInvalidValue;
  const GemvPlan p = gemv_plan(a.N, a.K, a.epilogue == 0);
  if (a.ksplit != p.ksplit) return hipErrorInvalidValue;  // the caller sizes its slots from the same plan
  const dim3 grid(a.N / 16 / p.tn, a.ksplit), block(p.waves * 64);
  if (p.waves == 8 && p.tn == 2) hipLaunchKernelGGL((gemv_mfma_kernel<8, 2, 2>), grid, block, 0, s, a);
  else if (p.waves == 8) hipLaunchKernelGGL((gemv_mfma_kernel<8, 2, 4>), grid, block, 0, s, a);
  else if (p.tn == 4) hipLaunchKernelGGL((gemv_mfma_kernel<4, 2, 4>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gemv_mfma_kernel<4, 4, 2>), grid, block, 0, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Decode attention.  Workgroup (split, kv head, sequence): the positions are cut into at most n_splits runs of a multiple
// of 128, computed from the position itself, so that the grid stays the same while the sequence grows; the 4 wavefronts
// take 32-key blocks of the run round robin, each with its own running softmax, and merge through LDS.  It is bound by
// the one pass over the cache: a wavefront requests the 16 KiB of a block at once, and the wavefronts beside it compute
// meanwhile (one register buffer, three wavefronts per SIMD; a second buffer for the next block left two and was slower:
// 8B shape, batch 64, 1024 positions, whole case 3248 -> 2939 us, batch 40 2633 -> 2285, 70B R = 8 batch 64 2047 -> 1969; 1.2B
// batch 32 1544 -> 1561).  All on the matrix cores, transposed so that nothing is shuffled:
//   S^T[key][column] = K Q^T     A = 16 keys x 32 dims, straight from the K rows (row i of tile t is key 8 (i / 4) + 4 t +
//                                i % 4 of the block, so that a lane ends up with eight neighbouring keys and its share of
//                                V^T is 16 contiguous bytes); B: the q heads of the group twice, in columns 0..7 and 8..15;
//   O^T[dim][column] = V^T P^T   A = 16 dims x 32 keys from the transposed V cache; B = the lane's own eight
//                                probabilities, split: their bf16 rounding in columns 0..7 and what it left out, rounded in
//                                turn, in 8..15 (16 significant bits); the two halves of O^T are added at the end.
// With one split the workgroup writes the output, else the splits' (max, sum, unnormalised output) go to the combine kernel.
// 64 sequences x 8 kv heads x 4 q heads x 1024 positions: 82 us + 9 for the combine -> 61 us by itself (4.4 TB/s).  (Vector units and chunks
// of 128 positions before.)
// ------------------------------------------------------------------------------------------------
__host__ __device__ __forceinline__ int attn_split_len(int n_pos, int n_splits) { return ((n_pos + n_splits - 1) / n_splits + 127) / 128 * 128; }

template <int D, int G>
__global__ __launch_bounds__(256, 3) void attn_decode_kernel(AttnDecodeArgs a) {
  constexpr int DS = D / 32, DT = D / 16;
  __shared__ float osm[4][G][D];
  __shared__ float msm[4][G], lsm[4][G];
  const int c = blockIdx.x, kvh = blockIdx.y, bi = blockIdx.z;
  const int n_pos = a.pos_dev ? (*a.pos_dev + 1) : a.n_pos;
  const int len = attn_split_len(n_pos, a.n_splits);
  const int p0 = c * len, p1 = min(n_pos, p0 + len);
  if (p0 >= p1) return;   // (the combine kernel looks at the splits that hold positions only)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = lane & 15, q = lane >> 4;
  const int nb = (p1 - p0 + 31) >> 5;
  const float scale = 1.0f / sqrtf((float)D);
  const int head = min(b & 7, G - 1);   // (columns without a head repeat one: finite, never stored)
  const bf16_t* qg = a.q + (size_t)bi * a.nq * D + (size_t)(kvh * G + head) * D;
  const bf16_t* kb = a.cache_k + (((size_t)bi * a.nkv + kvh) * a.max_seq + p0 + 8 * (b >> 2) + (b & 3)) * D + q * 8;
  const bf16_t* vb = a.cache_v + (((size_t)bi * a.nkv + kvh) * D + b) * a.max_seq + p0 + 8 * q;
  u32x4_t qr[DS];
#pragma unroll
  for (int s = 0; s < DS; ++s) qr[s] = *reinterpret_cast<const u32x4_t*>(qg + s * 32 + q * 8);

  f32x4_t o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) o[t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  struct Block { u32x4_t k[2][DS], v[DT]; };
  auto load = [&](Block& x, int blk) {   // (whole blocks: the capacity is a multiple of 32)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int s = 0; s < DS; ++s)
        x.k[t][s] = *reinterpret_cast<const u32x4_t*>(kb + (size_t)(blk * 32 + 4 * t) * D + s * 32);
#pragma unroll
    for (int t = 0; t < DT; ++t)
      x.v[t] = *reinterpret_cast<const u32x4_t*>(vb + (size_t)t * 16 * a.max_seq + blk * 32);
  };
  auto compute = [&](Block& x, int blk) {
    const int ahead = p1 - (p0 + blk * 32);
    if (ahead < 32) {   // (uniform) the run's last block: a probability of 0 does not cancel an infinity or NaN that an earlier,
                        // longer sequence left behind the run, so the V entries of the lane's keys ahead - 8 q .. 7 are cleared
      const int keep = ahead - 8 * q;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t mask = (2 * e < keep ? 0x0000FFFFu : 0u) | (2 * e + 1 < keep ? 0xFFFF0000u : 0u);
          x.v[t][e] &= mask;
        }
    }
    f32x4_t st[2];
    float sv[8], mloc = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      st[t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < DS; ++s)
        st[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x.k[t][s]), __builtin_bit_cast(bf16x8_t, qr[s]), st[t], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float v = p0 + blk * 32 + 8 * q + 4 * t + r < p1 ? st[t][r] * scale : -INFINITY;
        sv[t * 4 + r] = v;
        mloc = fmaxf(mloc, v);
      }
    }
    mloc = fmaxf(mloc, __shfl_xor(mloc, 16, 64));
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float mnew = fmaxf(m, mloc);
    const float ref = mnew == -INFINITY ? 0.f : mnew;   // (scores that are all -inf weigh nothing, they must not become NaN)
    const float corr = __expf(m - ref);
    float psum = 0.f;
    uint32_t pk[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float part[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float p = __expf(sv[2 * e + h] - ref);
        psum += p;
        const float high = bf16_to_f32(f32_to_bf16(p));
        part[h] = b < 8 ? high : p - high;
      }
      pk[e] = (uint32_t)f32_to_bf16(part[0]) | ((uint32_t)f32_to_bf16(part[1]) << 16);
    }
    l = l * corr + psum;
    m = mnew;
    const u32x4_t pb = {pk[0], pk[1], pk[2], pk[3]};
#pragma unroll
    for (int t = 0; t < DT; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o[t][r] *= corr;
      o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x.v[t]), __builtin_bit_cast(bf16x8_t, pb), o[t], 0, 0, 0);
    }
  };
  for (int blk = wave; blk < nb; blk += 4) {
    Block x;
    load(x, blk);
    __builtin_amdgcn_sched_barrier(0);
    compute(x, blk);
    __builtin_amdgcn_sched_barrier(0);
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = o[t][r] + __shfl_xor(o[t][r], 8, 64);
      if (b < G) osm[wave][b][t * 16 + 4 * q + r] = v;
    }
  if (q == 0 && b < G) { msm[wave][b] = m; lsm[wave][b] = l; }
  __syncthreads();
  const size_t part = (((size_t)bi * a.nkv + kvh) * a.n_splits + c) * G;
  for (int i = tid; i < G * D; i += 256) {
    const int h = i / D, dim = i % D;
    float mm = msm[0][h];   // (wavefront 0 always has a block)
#pragma unroll
    for (int w = 1; w < 4; ++w) mm = fmaxf(mm, msm[w][h]);
    const float ref = mm == -INFINITY ? 0.f : mm;
    float ll = 0.f, oo = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float e = __expf(msm[w][h] - ref);
      ll += lsm[w][h] * e;
      oo += osm[w][h][dim] * e;
    }
    if (a.n_splits == 1) {
      a.o[(size_t)bi * a.nq * D + (size_t)(kvh * G + h) * D + dim] = f32_to_bf16(oo / ll);
    } else {
      a.part_o[(part + h) * D + dim] = oo;
      if (dim == 0) {
        a.part_ml[(part + h) * 2 + 0] = mm;
        a.part_ml[(part + h) * 2 + 1] = ll;
      }
    }
  }
}

// combine: one workgroup of D threads per (sequence, q head); the splits' statistics go through LDS
// so that no thread walks a chain of dependent global loads
template <int D>
__global__ void attn_combine_kernel(AttnDecodeArgs a) {
  __shared__ float wgt[ATTN_DECODE_MAX_SPLITS];
  __shared__ float stat[2];
  const int h = blockIdx.x, bi = blockIdx.y, t = threadIdx.x;
  const int g = a.nq / a.nkv;
  const int kvh = h / g, hg = h % g;
  const int n_pos = a.pos_dev ? (*a.pos_dev + 1) : a.n_pos;
  const int len = attn_split_len(n_pos, a.n_splits);
  const int nc = (n_pos + len - 1) / len;   // splits that hold visible positions
  const size_t base = ((size_t)bi * a.nkv + kvh) * a.n_splits;
  for (int c = t; c < nc; c += D) wgt[c] = a.part_ml[((base + c) * g + hg) * 2];
  __syncthreads();
  if (t < 64) {   // first wavefront: max, then weights and the normaliser
    float m = -INFINITY;
    for (int c = t; c < nc; c += 64) m = fmaxf(m, wgt[c]);
    m = wave_max(m);
    float l = 0.f;
    for (int c = t; c < nc; c += 64) {
      const float w = __expf(wgt[c] - m);
      wgt[c] = w;
      l += a.part_ml[((base + c) * g + hg) * 2 + 1] * w;
    }
    l = wave_sum(l);
    if (t == 0) stat[0] = l;
  }
  __syncthreads();
  float o = 0.f;
#pragma unroll 8
  for (int c = 0; c < nc; ++c) o += a.part_o[((base + c) * g + hg) * D + t] * wgt[c];
  a.o[(size_t)bi * a.nq * D + h * D + t] = f32_to_bf16(o / stat[0]);
}

// splits of a (sequence, kv head): as many as give the chip (256 CUs) two workgroups per CU and no more (a few workgroups of a second
// round cost a round), of at least 128 positions each
int attn_decode_splits(int B, int nkv, int max_seq) {
  const int want = 512 / (B * nkv), most = (max_seq + 127) / 128;
  const int n = want < 1 ? 1 : want < most ? want : most;
  return n < ATTN_DECODE_MAX_SPLITS ? n : ATTN_DECODE_MAX_SPLITS;
}

template <int D, int G>
static hipError_t launch_attn_decode_t(const AttnDecodeArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((attn_decode_kernel<D, G>), dim3(a.n_splits, a.nkv, a.B), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_splits == 1) return e;
  hipLaunchKernelGGL(attn_combine_kernel<D>, dim3(a.nq, a.B), dim3(D), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_attn_decode(const AttnDecodeArgs& a, hipStream_t s) {
  if (a.n_splits < 1 || a.n_splits > ATTN_DECODE_MAX_SPLITS || (a.max_seq & 31)) return hipErrorInvalidValue;
  const int g = a.nq / a.nkv;
  if (a.d == 128) {
    switch (g) {
      case 1: return launch_attn_decode_t<128, 1>(a, s);
      case 2: return launch_attn_decode_t<128, 2>(a, s);
      case 4: return launch_attn_decode_t<128, 4>(a, s);
      case 8: return launch_attn_decode_t<128, 8>(a, s);
    }
  } else if (a.d == 64) {
    switch (g) {
      case 1: return launch_attn_decode_t<64, 1>(a, s);
      case 2: return launch_attn_decode_t<64, 2>(a, s);
      case 4: return launch_attn_decode_t<64, 4>(a, s);
      case 8: return launch_attn_decode_t<64, 8>(a, s);
    }
  }
  return hipErrorInvalidValue;
}
