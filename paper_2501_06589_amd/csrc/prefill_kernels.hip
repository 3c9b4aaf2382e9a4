// Prefill-shape kernels of the bf16 path (gfx950): MFMA GEMM on the packed weight tiles and causal
// GQA flash attention over the cache, both on v_mfma_f32_16x16x32_bf16.
#include "common.h"
#include "gemm_choice.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;

__device__ __forceinline__ void unpack8(const uint4 v, float (&f)[8]) {
  f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
  f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
  f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xFFFF0000u);
  f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xFFFF0000u);
}

__device__ __forceinline__ f32x4_t mfma16(const uint4 a, const uint4 b, const f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}

// ------------------------------------------------------------------------------------------------
// C[M][N] = X[M][K] W[K][N] on the packed weight tiles: three kernels, gemm_duo_kernel (128 rows, two workgroups per CU) for many
// rows, gemm_lds_kernel (256 x 256 tiles, one per CU) for the shapes where it stays ahead of that, and gemm_ring_kernel (smaller
// tiles, a deep queue of weights) for few rows and odd K; gemm_best_tile chooses.
// In all of them the weights are the MFMA A operand and the activations the B operand, so output element (m, n) sits in
// lane (n%16)/4*16 + m%16, register n%4: a lane stores 4 consecutive columns.
// Rows >= M and weight tiles >= N/16 are clamped on load: they only reach outputs that are not stored.
// ------------------------------------------------------------------------------------------------
// Epilogue of a wavefront's (16 JT)-column x (16 WM)-row accumulator block: row base m0, first weight tile nt0.
// Output element (m, n) sits in lane (n%16)/4*16 + m%16, register n%4: a lane stores 4 consecutive columns.
// RESIDUAL: epilogue 3 is among those the kernel takes (the tiles of 192 columns and more update the residual through LDS, 64 x 64 ones never do).
template <int WM, int JT, bool RESIDUAL>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, f32x4_t (&acc)[JT][WM], int m0, int nt0, int NT, int lane) {
  const int b = lane & 15, q = lane >> 4;
  // row scale (1.0 where there is none: the multiplication is exact then), applied where an accumulator is read
  auto scale_of = [&](int mt) { return a.row_scale ? a.row_scale[min(m0 + mt * 16 + b, a.M - 1)] : 1.0f; };
  if constexpr (RESIDUAL) {
    static_assert(JT % 2 == 0, "two column tiles at a time");
    if (a.epilogue == 3) {
      // residual update; the summation order per element is fixed: old value, product, peers 0, 1, ...
      // The operands (old values, the first three peers) of two column tiles are requested at once.
      constexpr int PB = 3, JB = 2, JG = JT / JB, STEPS = WM * JG;
      struct Operands { float4 xo[JB]; uint2 pk[JB][PB]; };
      Operands o;
      auto row_of = [&](int mt) { return (size_t)min(m0 + mt * 16 + b, a.M - 1) * a.N; };
      auto request = [&](Operands& o, int st) {
        const size_t row = row_of(st / JG);
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
          const size_t off = row + min(nt0 + (st % JG) * JB + jj, NT - 1) * 16 + 4 * q;
          if (a.x_emb) {
            const uint2 e = *reinterpret_cast<const uint2*>(a.x_emb + off);
            o.xo[jj] = __builtin_bit_cast(float4, make_uint4(e.x << 16, e.x & 0xFFFF0000u, e.y << 16, e.y & 0xFFFF0000u));
          } else {
            o.xo[jj] = *reinterpret_cast<const float4*>(a.x_res + off);
          }
#pragma unroll
          for (int p = 0; p < PB; ++p)
            if (p < a.n_peers) o.pk[jj][p] = *reinterpret_cast<const uint2*>(a.peers + p * a.peer_stride + off);
        }
      };
      auto add_peer = [&](float (&v4)[4], const uint2 pk) {
        v4[0] += __uint_as_float(pk.x << 16);
        v4[1] += __uint_as_float(pk.x & 0xFFFF0000u);
        v4[2] += __uint_as_float(pk.y << 16);
        v4[3] += __uint_as_float(pk.y & 0xFFFF0000u);
      };
      float ss = 0.f;
#pragma unroll
      for (int st = 0; st < STEPS; ++st) {
        request(o, st);
        const int mt = st / JG;
        const int m = m0 + mt * 16 + b;
        const bool ok = m < a.M;
        const size_t row = row_of(mt);
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
          const int j = (st % JG) * JB + jj;
          if (nt0 + j >= NT) continue;   // (uniform over the wavefront)
          const size_t off = row + (nt0 + j) * 16 + 4 * q;
          float v4[4] = {o.xo[jj].x + acc[j][mt][0], o.xo[jj].y + acc[j][mt][1], o.xo[jj].z + acc[j][mt][2], o.xo[jj].w + acc[j][mt][3]};
#pragma unroll
          for (int p = 0; p < PB; ++p)
            if (p < a.n_peers) add_peer(v4, o.pk[jj][p]);
          for (int p = PB; p < a.n_peers; ++p) add_peer(v4, *reinterpret_cast<const uint2*>(a.peers + p * a.peer_stride + off));
          if (ok) {
            if (!a.last) *reinterpret_cast<float4*>(a.x_res + off) = make_float4(v4[0], v4[1], v4[2], v4[3]);
            if (a.x_copy)
              *reinterpret_cast<float4*>(a.x_copy + off) = a.copy_step ? make_float4(v4[0] - o.xo[jj].x, v4[1] - o.xo[jj].y, v4[2] - o.xo[jj].z, v4[3] - o.xo[jj].w)
                                                                       : make_float4(v4[0], v4[1], v4[2], v4[3]);
            // the rows as the modules that read them want them: times their norm's gain (fp32 product, one rounding)
            auto store_gained = [&](bf16_t* dst, const bf16_t* gain) {
              const uint2 gk = *reinterpret_cast<const uint2*>(gain + (nt0 + j) * 16 + 4 * q);
              const float g4[4] = {__uint_as_float(gk.x << 16), __uint_as_float(gk.x & 0xFFFF0000u),
                                   __uint_as_float(gk.y << 16), __uint_as_float(gk.y & 0xFFFF0000u)};
              uint2 pk;
              pk.x = f32_to_bf16x2(v4[0] * g4[0], v4[1] * g4[1]);
              pk.y = f32_to_bf16x2(v4[2] * g4[2], v4[3] * g4[3]);
              *reinterpret_cast<uint2*>(dst + off) = pk;
            };
            if (a.xh_a) store_gained(a.xh_a, a.gain_a);
            if (a.xh_b) store_gained(a.xh_b, a.gain_b);
          }
          ss += v4[0] * v4[0] + v4[1] * v4[1] + v4[2] * v4[2] + v4[3] * v4[3];
        }
        if (st % JG == JG - 1) {   // the row block is complete: its rows' sums of squares over this wavefront's columns
          ss += __shfl_xor(ss, 16, 64);
          ss += __shfl_xor(ss, 32, 64);
          if (a.ssq_part && q == 0 && ok && nt0 < NT) a.ssq_part[(size_t)(nt0 / JT) * a.M + m] = ss;
          ss = 0.f;
        }
      }
      return;
    }
  }
  if (a.epilogue == 0) {
#pragma unroll
    for (int mt = 0; mt < WM; ++mt) {
      const int m = m0 + mt * 16 + b;
      const float rs = scale_of(mt);
      if (m >= a.M) continue;
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        if (nt0 + j >= NT) continue;
        const int n = (nt0 + j) * 16 + 4 * q;
        *reinterpret_cast<float4*>(a.out + (size_t)m * a.N + n) =
            make_float4(acc[j][mt][0] * rs, acc[j][mt][1] * rs, acc[j][mt][2] * rs, acc[j][mt][3] * rs);
      }
    }
  } else if (a.epilogue == 2) {
    // rotary embedding + cache append: a lane's 4 columns are two adjacent pairs of one head
    const int half = a.d >> 1;
#pragma unroll
    for (int mt = 0; mt < WM; ++mt) {
      const int m = m0 + mt * 16 + b;
      const float rs = scale_of(mt);
      if (m >= a.M) continue;
      const int seq = m / a.T, pos = a.pos0 + m % a.T;
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        if (nt0 + j >= NT) continue;
        const int col = (nt0 + j) * 16 + 4 * q;
        const int head = col / a.d, dim = col % a.d;
        float v4[4] = {acc[j][mt][0] * rs, acc[j][mt][1] * rs, acc[j][mt][2] * rs, acc[j][mt][3] * rs};
        if (head < a.nq + a.nkv) {
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const float c = a.cos_tab[(size_t)pos * half + (dim >> 1) + p], sn = a.sin_tab[(size_t)pos * half + (dim >> 1) + p];
            const float e = v4[2 * p], o = v4[2 * p + 1];
            v4[2 * p] = e * c - o * sn;
            v4[2 * p + 1] = e * sn + o * c;
          }
        }
        if (head < a.nq + a.nkv) {
          uint2 pk;
          pk.x = f32_to_bf16x2(v4[0], v4[1]);
          pk.y = f32_to_bf16x2(v4[2], v4[3]);
          bf16_t* dst = head < a.nq ? a.q_out + (size_t)m * a.nq * a.d + head * a.d + dim
                                    : a.cache_k + (((size_t)seq * a.nkv + (head - a.nq)) * a.max_seq + pos) * a.d + dim;
          *reinterpret_cast<uint2*>(dst) = pk;
        } else {
          bf16_t* vt = a.cache_v + (((size_t)seq * a.nkv + (head - a.nq - a.nkv)) * a.d + dim) * a.max_seq + pos;
#pragma unroll
          for (int r = 0; r < 4; ++r) vt[(size_t)r * a.max_seq] = f32_to_bf16(v4[r]);
          if (m % a.T == a.T - 1)
            for (int r = 0; r < 4; ++r) clear_block(vt + (size_t)r * a.max_seq + 1, pos + 1, a.max_seq);
        }
      }
    }
  } else {
    // SwiGLU: tile columns 0..7 = gate columns 8nt..8nt+7 (lanes q = 0, 1), columns 8..15 = the matching
    // up columns (lanes q = 2, 3): lane + 32 holds the up partner of this lane's gate value.
    const int I = a.N >> 1;
#pragma unroll
    for (int mt = 0; mt < WM; ++mt) {
      const int m = m0 + mt * 16 + b;
      const float rs = scale_of(mt);   // (lane + 32 holds the same row)
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        float r4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float g = acc[j][mt][r] * rs;
          const float u = __shfl(g, (lane + 32) & 63, 64);
          r4[r] = g / (1.0f + __expf(-g)) * u;
        }
        if (q < 2 && m < a.M && nt0 + j < NT) {
          uint2 pk;
          pk.x = f32_to_bf16x2(r4[0], r4[1]);
          pk.y = f32_to_bf16x2(r4[2], r4[3]);
          *reinterpret_cast<uint2*>(a.act + (size_t)m * I + (nt0 + j) * 8 + 4 * q) = pk;
        }
      }
    }
  }
}

// 64 rows per workgroup, the partial sums dealt out over its 16 wavefronts (a serial chain of loads otherwise: 64 parts x
// 2048 rows 17 us); fixed order: every wavefront its parts in turn, then the wavefronts 0 .. 15
__global__ __launch_bounds__(1024) void row_rms_kernel(const float* __restrict__ part, int n_part, int M, float h, float eps,
                                                       float* __restrict__ rs_a, float* __restrict__ rs_b) {
  __shared__ float sum[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = blockIdx.x * 64 + lane;
  float tot = 0.f;
  if (m < M) {
#pragma unroll 4
    for (int p = wave; p < n_part; p += 16) tot += part[(size_t)p * M + m];
  }
  sum[wave][lane] = tot;
  __syncthreads();
  if (wave > 0 || m >= M) return;
  tot = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) tot += sum[w][lane];
  const float rs = 1.0f / sqrtf(tot / h + eps);
  rs_a[m] = rs;
  if (rs_b) rs_b[m] = rs;
}

hipError_t launch_row_rms(const float* ssq_part, int n_part, int M, int H, float eps, float* rs_a, float* rs_b, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  hipLaunchKernelGGL(row_rms_kernel, dim3((M + 63) / 64), dim3(1024), 0, s, ssq_part, n_part, M, (float)H, eps, rs_a, rs_b);
  return hipGetLastError();
}

#define GEMM_GROUP_M 8   // row blocks that share one column block back to back
#define GEMM_EPI_STRIDE(bn) ((bn) + 4)   // floats per staged row of the residual epilogue
#define GEMM2_LDSP(p) ((__attribute__((address_space(3))) void*)(p))
#define GEMM2_GLBP(p) ((const __attribute__((address_space(1))) void*)(p))

// s_waitcnt vmcnt(N) lgkmcnt(0): this wave's LDS reads are complete and at most N of its vector-memory operations in flight (gfx9
// encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8); then a bare workgroup barrier, without the fence of
// __syncthreads(), which would wait for ALL outstanding loads.  Builtins, not inline assembly: after an asm statement the compiler
// no longer knows which LDS reads are pending and waits for all of them at the next use.
template <int N>
__device__ __forceinline__ void ring_meet() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// 16 bytes that no cache should keep
__device__ __forceinline__ uint4 load_once(const void* p) {
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p)));
}

// the staged column that lane l of a row reads (192 columns: 24 of the 32 lanes have eight each, the others repeat the first)
template <int BN>
__device__ __forceinline__ constexpr int gemm_staged_column(int l) { return 8 * l < BN ? 8 * l : 0; }

// Epilogue 3 of a workgroup's tile of WR x 16 MT rows and WC x 16 JT columns (see GemmArgs), with whole rows per memory
// instruction.  In the accumulator layout a wavefront's load or store touches 16 rows, 64 (fp32) or 32 (bf16) bytes of each, and
// in that shape the 16 - 26 bytes per element that the update moves cost as much as a reduce kernel of its own.  So the tile
// passes through LDS (free once the workgroup is past its last k tile), 64 rows at a time: the wavefronts write their accumulator
// blocks, meet, and read back one row of the tile per half-wavefront (quarter, for 128 columns), eight columns per lane: 16 bytes
// per lane and instruction, row segments of 512 bytes and more.  The rows' sums of squares are left per column block of the tile:
// ssq_part[n_blk][m].  The summation order per element is fixed: old value, product, peers 0, 1, ...
// The peers are read once per call and bypass the caches (non-temporal): they would push out the operands that the workgroups
// beside are multiplying and the rows that the next kernels read (4001 x 8192, seven peers, K 1024 / 3584: 224 / 300 -> 188 / 277 us).
// (The rows themselves non-temporal too: 1 - 4 % faster measured alone where they exceed the last-level cache, no different in a call.)
template <int MT, int JT, int WR, int WC, int PB>   // PB: peers requested at once (0: there are none)
__device__ __forceinline__ void gemm_residual_epilogue(const GemmArgs& a, f32x4_t (&acc)[JT][MT], unsigned char* lds, int m0,
                                                       int n_blk, int wave, int lane) {
  constexpr int BN = 16 * JT * WC, STRIDE = GEMM_EPI_STRIDE(BN);   // floats per staged row: + 4, so that the 16 rows of a write spread over the banks
  constexpr int LPR = BN > 128 ? 32 : 16, RPI = 64 / LPR;          // lanes per row, rows per instruction
  constexpr int ROWS = 64 / WR, H = ROWS / 16;                     // staged rows and row tiles per wavefront row and pass
  constexpr int STEPS = 64 / (WR * WC * RPI);                      // rows that a lane group takes per pass
  constexpr int RB = 2;                                            // rows requested at once
  static_assert(STEPS % RB == 0 && MT % H == 0, "whole passes");
  static_assert(gemm_staged_column<BN>(LPR - 1) + 8 <= STRIDE, "the lanes of a row read inside it");
  float* stage = reinterpret_cast<float*>(lds);
  const int b = lane & 15, q = lane >> 4, wr = wave / WC, wc = wave % WC;
  const int sub = lane / LPR, l = lane % LPR;
  const int n = n_blk * BN + 8 * l;
  const bool col_ok = 8 * l < BN && n < a.N;   // (N is a multiple of 16)
  const int nc = col_ok ? n : 0;
  const int lc = gemm_staged_column<BN>(l);
  // the gains of the modules that read the new rows, for this lane's eight columns (the same for every row)
  float ga8[8], gb8[8];
  unpack8(a.xh_a ? *reinterpret_cast<const uint4*>(a.gain_a + nc) : make_uint4(0, 0, 0, 0), ga8);
  unpack8(a.xh_b ? *reinterpret_cast<const uint4*>(a.gain_b + nc) : make_uint4(0, 0, 0, 0), gb8);
#pragma unroll
  for (int pass = 0; pass < MT / H; ++pass) {
    if (pass > 0) __syncthreads();           // the previous pass has been read
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int j = 0; j < JT; ++j)
        *reinterpret_cast<f32x4_t*>(stage + (wr * ROWS + h * 16 + b) * STRIDE + (wc * JT + j) * 16 + 4 * q) = acc[j][H * pass + h];
    __syncthreads();
#pragma unroll
    for (int g = 0; g < STEPS / RB; ++g) {
      float4 xo[RB][2];
      uint4 pk[RB][PB > 0 ? PB : 1];
      size_t off[RB];
      bool ok[RB];
      int mrow[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int lr = ((g * RB + r) * (WR * WC) + wave) * RPI + sub;   // staged row
        mrow[r] = m0 + lr / ROWS * (MT * 16) + pass * ROWS + lr % ROWS;
        ok[r] = col_ok && mrow[r] < a.M;
        off[r] = (size_t)min(mrow[r], a.M - 1) * a.N + nc;
        if (a.x_emb) {
          xo[r][0] = __builtin_bit_cast(float4, load_16_at_8(a.x_emb + off[r]));
        } else {
          xo[r][0] = *reinterpret_cast<const float4*>(a.x_res + off[r]);
          xo[r][1] = *reinterpret_cast<const float4*>(a.x_res + off[r] + 4);
        }
#pragma unroll
        for (int p = 0; p < PB; ++p)
          if (p < a.n_peers) pk[r][p] = load_once(a.peers + p * a.peer_stride + off[r]);
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int lr = ((g * RB + r) * (WR * WC) + wave) * RPI + sub;
        const float4 p0 = *reinterpret_cast<const float4*>(stage + lr * STRIDE + lc);
        const float4 p1 = *reinterpret_cast<const float4*>(stage + lr * STRIDE + lc + 4);
        float old8[8] = {xo[r][0].x, xo[r][0].y, xo[r][0].z, xo[r][0].w, xo[r][1].x, xo[r][1].y, xo[r][1].z, xo[r][1].w};
        if (a.x_emb) unpack8(__builtin_bit_cast(uint4, xo[r][0]), old8);
        float v8[8] = {old8[0] + p0.x, old8[1] + p0.y, old8[2] + p0.z, old8[3] + p0.w, old8[4] + p1.x, old8[5] + p1.y, old8[6] + p1.z, old8[7] + p1.w};
        auto add_peer = [&](const uint4 u) {
          float f[8];
          unpack8(u, f);
#pragma unroll
          for (int e = 0; e < 8; ++e) v8[e] += f[e];
        };
#pragma unroll
        for (int p = 0; p < PB; ++p)
          if (p < a.n_peers) add_peer(pk[r][p]);
        if constexpr (PB > 0)
          for (int p = PB; p < a.n_peers; ++p) add_peer(load_once(a.peers + p * a.peer_stride + off[r]));
        if (ok[r]) {
          if (!a.last) {
            *reinterpret_cast<float4*>(a.x_res + off[r]) = make_float4(v8[0], v8[1], v8[2], v8[3]);
            *reinterpret_cast<float4*>(a.x_res + off[r] + 4) = make_float4(v8[4], v8[5], v8[6], v8[7]);
          }
          if (a.x_copy) {
            if (!a.copy_step) {
#pragma unroll
              for (int e = 0; e < 8; ++e) old8[e] = 0.f;
            }
            *reinterpret_cast<float4*>(a.x_copy + off[r]) = make_float4(v8[0] - old8[0], v8[1] - old8[1], v8[2] - old8[2], v8[3] - old8[3]);
            *reinterpret_cast<float4*>(a.x_copy + off[r] + 4) = make_float4(v8[4] - old8[4], v8[5] - old8[5], v8[6] - old8[6], v8[7] - old8[7]);
          }
          // the rows as the modules that read them want them: times their norm's gain (fp32 product, one rounding)
          auto store_gained = [&](bf16_t* dst, const float (&g8)[8]) {
            uint4 u;
            u.x = f32_to_bf16x2(v8[0] * g8[0], v8[1] * g8[1]);
            u.y = f32_to_bf16x2(v8[2] * g8[2], v8[3] * g8[3]);
            u.z = f32_to_bf16x2(v8[4] * g8[4], v8[5] * g8[5]);
            u.w = f32_to_bf16x2(v8[6] * g8[6], v8[7] * g8[7]);
            *reinterpret_cast<uint4*>(dst + off[r]) = u;
          };
          if (a.xh_a) store_gained(a.xh_a, ga8);
          if (a.xh_b) store_gained(a.xh_b, gb8);
        }
        if (a.ssq_part) {   // (uniform)
          float ss = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) ss += v8[e] * v8[e];
          if (!ok[r]) ss = 0.f;
#pragma unroll
          for (int o = LPR / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);   // over the lanes of the row
          if (l == 0 && mrow[r] < a.M) a.ssq_part[(size_t)n_blk * a.M + mrow[r]] = ss;
        }
      }
    }
  }
}

// dynamic LDS above the default 64 KiB has to be allowed per kernel and device, once
static hipError_t allow_lds(const void* kernel, int bytes, bool (&prepared)[64]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!prepared[dev]) {
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    prepared[dev] = true;
  }
  return hipSuccess;
}

// ------------------------------------------------------------------------------------------------
// Large-M GEMM: 256 x 256 workgroup tile, 8 wavefronts (2 along M x 4 along N, 128 x 64 each), one
// workgroup per CU.  Both operands travel global memory -> LDS without passing through registers
// (16-byte direct-to-LDS loads: the 64 lanes of one load fill 1 KiB of LDS in lane order), so loads are
// in flight two to three k tiles ahead of the MFMAs that consume them and cost no registers.
//   Weights: a ring of 4 stages of one k tile (32): 16 packed tiles of 1 KiB, each the register image of
//   an MFMA operand (read back as one contiguous 1 KiB).
//   Activations: a ring of 3 blocks of TWO k tiles (256 rows x 128 bytes): one load covers 8 rows x 64 k,
//   i.e. whole 128-byte cache lines (a load of 16 rows x 32 k would request every line twice, half a line
//   per k tile: measured 4 - 7 % slower).  Within a block the 16-byte segments of fragment row b are
//   stored XOR-swizzled by b / 2 (the lane that fetches segment s of row b sits at position s ^ (b / 2) of
//   the row's eight lanes), so that the 16 lanes of a fragment read that hold the same k segment hit 16
//   different bank groups.
// 160 KiB of LDS in all.  One bare barrier per k tile, in the middle of its MFMAs: after the barrier of k
// tile kt every wave's loads for k tile kt + 1 have landed and every wave has finished reading k tile
// kt - 1, whose buffers the next loads overwrite.  The first fragments of k tile kt + 1 are read right
// after that barrier, sixteen MFMAs before their first use, and a wave's loads are spread over its MFMA
// rows (issued in one burst by all eight waves they fill the address pipeline, and a wave that cannot
// issue its load cannot issue the MFMAs behind it either).
// Rows >= M and weight tiles >= N/16 are clamped on load (they only reach outputs that are not stored).
// K must be a multiple of 64.
// Tile order: workgroups are handed to the 8 XCDs round robin by block index and every XCD has its own L2, so block
// index i is mapped to position (i % 8) * (n / 8) + i / 8 of the tile order: each XCD works through one contiguous
// eighth of it and neighbours in the order (which share operands) meet in one L2.  GEMM2_GROUP_M row blocks share one
// column block back to back; the 32 CUs of an XCD then work on 4 row blocks x 8 column blocks at a time (groups of 2 / 4 / 8 row blocks:
// 1309 / 1335 / 1297 TFLOP/s on 32768 x 8192 x 14336 with SwiGLU, which gemm_duo_kernel now takes at 1414).
// What it takes (gemm_choice.h; of the configured shapes): QKV of thousands of rows (32768 x 2560 x 8192: 1177 - 1222 TFLOP/s), residual updates without
// peers of 4000 rows and more (8B shape, 8192 rows, O + down 962 us in place, gemm_duo_kernel 1030) and SwiGLU of some calls of 385 - 1024 rows
// (400 x 28672 x 4096 111 us, 125).
// ------------------------------------------------------------------------------------------------
#define GEMM2_GROUP_M 4
// as ring_meet, but the LDS reads in flight are left alone
template <int N>
__device__ __forceinline__ void gemm2_wait_and_meet() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

#define GEMM2_XBLOCK_BYTES 32768
#define GEMM2_WSTAGE_BYTES 16384
#define GEMM2_XBLOCKS 3
#define GEMM2_WSTAGES 4
#define GEMM2_LDS_BYTES (GEMM2_XBLOCKS * GEMM2_XBLOCK_BYTES + GEMM2_WSTAGES * GEMM2_WSTAGE_BYTES)

__global__ __launch_bounds__(512, 2) void gemm_lds_kernel(GemmArgs a) {
  constexpr int WM = 8;
  extern __shared__ __attribute__((aligned(16))) unsigned char g2_lds[];
  unsigned char* const xring = g2_lds;
  unsigned char* const wring = g2_lds + GEMM2_XBLOCKS * GEMM2_XBLOCK_BYTES;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = lane & 15, q = lane >> 4;
  const int wm = wave >> 2, wn = wave & 3;
  const int KT = a.K >> 5, KB = a.K >> 6, NT = a.N >> 4;
  const int tiles_m = (a.M + 255) / 256, tiles_n = (a.N + 255) / 256;
  const int nblk = gridDim.x, nblk8 = nblk & ~7;   // XCD-aware order
  const int bid = (int)blockIdx.x < nblk8 ? ((int)blockIdx.x & 7) * (nblk8 >> 3) + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
  const int per_group = GEMM2_GROUP_M * tiles_n;
  const int group = bid / per_group, in_group = bid % per_group;
  const int gm = min(GEMM2_GROUP_M, tiles_m - group * GEMM2_GROUP_M);
  const int m_blk = group * GEMM2_GROUP_M + in_group % gm;
  const int n_blk = in_group / gm;
  const int m0 = m_blk * 256;
  const int nt0 = n_blk * 16;

  // this wave's share of the loads: row groups (8 rows) 4 wave .. 4 wave + 3 of an activation block, weight
  // tiles 2 wave, 2 wave + 1 of a stage
  const bf16_t* xsrc[4];
  const u32x4_t* wsrc[2];
  {
    const int r = lane >> 3;   // row within the group of 8
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int g = 4 * wave + i;                  // row group of the tile
      const int brow = 8 * (g & 1) + r;            // row within its 16-row fragment
      const int seg = (lane & 7) ^ ((brow >> 1) & 7);
      xsrc[i] = a.x + (size_t)min(m0 + 8 * g + r, a.M - 1) * a.ldx + seg * 8;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      wsrc[i] = reinterpret_cast<const u32x4_t*>(a.wp) + (size_t)min(nt0 + 2 * wave + i, NT - 1) * KT * 64 + lane;
  }
  auto issue_x = [&](int xbuf, int kb, int i) {   // row group i of this wave, activation block kb (k tiles 2 kb, 2 kb + 1)
    const int kbc = min(kb, KB - 1);
    __builtin_amdgcn_global_load_lds(GEMM2_GLBP(xsrc[i] + (size_t)kbc * 64),
                                     GEMM2_LDSP(xring + xbuf * GEMM2_XBLOCK_BYTES + (4 * wave + i) * 1024), 16, 0, 0);
  };
  auto issue_w = [&](int wbuf, int kt, int i) {   // weight tile i of this wave, k tile kt
    const int ktc = min(kt, KT - 1);
    __builtin_amdgcn_global_load_lds(GEMM2_GLBP(wsrc[i] + (size_t)ktc * 64),
                                     GEMM2_LDSP(wring + wbuf * GEMM2_WSTAGE_BYTES + (2 * wave + i) * 1024), 16, 0, 0);
  };

  f32x4_t acc[4][WM];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int mt = 0; mt < WM; ++mt) acc[j][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

  // per-lane read offsets inside an activation block, for the even and the odd k tile of the block
  const int xoff0 = (b >> 3) * 1024 + ((b & 7) * 8 + ((q) ^ ((b >> 1) & 7))) * 16 + wm * 8 * 2048;
  const int xoff1 = (b >> 3) * 1024 + ((b & 7) * 8 + ((4 + q) ^ ((b >> 1) & 7))) * 16 + wm * 8 * 2048;
  auto xfrag = [&](const unsigned char* xb, int mt) { return *reinterpret_cast<const u32x4_t*>(xb + mt * 2048); };
  auto wfrag = [&](const unsigned char* wb, int j) { return *reinterpret_cast<const u32x4_t*>(wb + (wn * 4 + j) * 1024); };
  auto mfma_row = [&](const u32x4_t (&w)[4], const u32x4_t& f, int mt) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[j]),
                                                          __builtin_bit_cast(bf16x8_t, f), acc[j][mt], 0, 0, 0);
  };

  // Issue order of a wave, per pair of k tiles (2j, 2j + 1); s = weight stage = k tile, blk = activation block:
  //   2j   first half : W1(s 2j+2)                       barrier 2j   needs W(2j+1)            -> vmcnt(4)
  //   2j   second half: W0(s 2j+3) X0 X1(blk j+2)
  //   2j+1 first half : W1(s 2j+3) X2 X3(blk j+2)        barrier 2j+1 needs W(2j+2), X(j+1)    -> vmcnt(6)
  //   2j+1 second half: W0(s 2j+4)
  // prologue in the same order: X(blk 0) W(0) | W0(1) X0 X1(blk 1) | W1(1) X2 X3(blk 1) | W0(2)
#pragma unroll
  for (int i = 0; i < 4; ++i) issue_x(0, 0, i);
  issue_w(0, 0, 0);
  issue_w(0, 0, 1);
  issue_w(1, 1, 0);
  issue_x(1, 1, 0);
  issue_x(1, 1, 1);
  issue_w(1, 1, 1);
  issue_x(1, 1, 2);
  issue_x(1, 1, 3);
  issue_w(2, 2, 0);
  gemm2_wait_and_meet<7>();   // block 0 and stage 0 have landed
  u32x4_t wA[4], wB[4], fA[3], fB[3];
#pragma unroll
  for (int j = 0; j < 4; ++j) wA[j] = wfrag(wring + lane * 16, j);
#pragma unroll
  for (int mt = 0; mt < 3; ++mt) fA[mt] = xfrag(xring + xoff0, mt);

  int wstage = 0;   // weight stage of the current k tile
  int xblk = 0;     // activation block of the current pair of k tiles
  // one k tile; ODD: second tile of its activation block
  auto step = [&](auto odd_tag, const u32x4_t (&w)[4], const u32x4_t (&f012)[3], u32x4_t (&wn4)[4], u32x4_t (&g012)[3], int kt) {
    constexpr bool ODD = decltype(odd_tag)::value;
    const unsigned char* xb = xring + xblk * GEMM2_XBLOCK_BYTES + (ODD ? xoff1 : xoff0);
    const int wnext = (wstage + 1) & 3, w2 = (wstage + 2) & 3, w3 = (wstage + 3) & 3;
    const int xnext = xblk + 1 == GEMM2_XBLOCKS ? 0 : xblk + 1;
    const int xfill = xblk + 2 >= GEMM2_XBLOCKS ? xblk + 2 - GEMM2_XBLOCKS : xblk + 2;
    u32x4_t f[WM];
    mfma_row(w, f012[0], 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mt = 3; mt < WM; ++mt) f[mt] = xfrag(xb, mt);
    __builtin_amdgcn_sched_barrier(0);
    mfma_row(w, f012[1], 1);
    __builtin_amdgcn_sched_barrier(0);
    if (ODD) {
      issue_w(w2, kt + 2, 1);
      issue_x(xfill, (kt >> 1) + 2, 2);
    } else {
      issue_w(w2, kt + 2, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    mfma_row(w, f012[2], 2);
    __builtin_amdgcn_sched_barrier(0);
    mfma_row(w, f[3], 3);
    __builtin_amdgcn_sched_barrier(0);
    if (ODD) issue_x(xfill, (kt >> 1) + 2, 3);
    __builtin_amdgcn_sched_barrier(0);
    // after the barrier: weight stage kt + 1 (and, behind an odd tile, the next activation block) are readable,
    // and nobody reads weight stage kt - 1 (behind an even tile: activation block j - 1) any more
    if (ODD) gemm2_wait_and_meet<6>(); else gemm2_wait_and_meet<4>();
    const unsigned char* nxb = ODD ? xring + xnext * GEMM2_XBLOCK_BYTES + xoff0 : xring + xblk * GEMM2_XBLOCK_BYTES + xoff1;
    const unsigned char* nwb = wring + wnext * GEMM2_WSTAGE_BYTES + lane * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) wn4[j] = wfrag(nwb, j);
#pragma unroll
    for (int mt = 0; mt < 3; ++mt) g012[mt] = xfrag(nxb, mt);
    __builtin_amdgcn_sched_barrier(0);
    mfma_row(w, f[4], 4);
    __builtin_amdgcn_sched_barrier(0);
    issue_w(w3, kt + 3, 0);
    if (!ODD) issue_x(xfill, (kt >> 1) + 2, 0);
    __builtin_amdgcn_sched_barrier(0);
    mfma_row(w, f[5], 5);
    mfma_row(w, f[6], 6);
    __builtin_amdgcn_sched_barrier(0);
    if (!ODD) issue_x(xfill, (kt >> 1) + 2, 1);
    __builtin_amdgcn_sched_barrier(0);
    mfma_row(w, f[7], 7);
    __builtin_amdgcn_sched_barrier(0);
    wstage = wnext;
    if (ODD) xblk = xnext;
  };
  for (int kt = 0; kt < KT; kt += 2) {   // KT is even
    step(std::false_type{}, wA, fA, wB, fB, kt);
    step(std::true_type{}, wB, fB, wA, fA, kt + 1);
  }
  // the clamped loads past the last k tile are still in flight into LDS: they must land before the workgroup ends
  gemm2_wait_and_meet<0>();
  if (a.epilogue == 3) gemm_residual_epilogue<WM, 4, 2, 4, 0>(a, acc, g2_lds, m0, n_blk, wave, lane);   // (calls with peers take other tiles)
  else gemm_epilogue<WM, 4, false>(a, acc, m0 + wm * 128, nt0 + wn * 4, NT, lane);
}

static hipError_t launch_gemm_lds(const GemmArgs& a, hipStream_t s) {
  static bool prepared[64] = {};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(gemm_lds_kernel), (int)GEMM2_LDS_BYTES, prepared);
  if (e != hipSuccess) return e;
  const int tiles_m = (a.M + 255) / 256, tiles_n = (a.N + 255) / 256;
  hipLaunchKernelGGL(gemm_lds_kernel, dim3(tiles_m * tiles_n), dim3(512), GEMM2_LDS_BYTES, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Many rows: 128 x 64 JT workgroup tile, 4 wavefronts side by side along N (128 rows x 16 JT columns each), two workgroups per CU.
// A wavefront shares its weight tiles with nobody, so they go from memory straight to registers, as packed (two stages of 64 k
// in flight, 64 registers at JT = 4); only the activations pass through LDS, a ring of DUO_STAGES stages of 64 k filled by
// direct-to-LDS loads.  A load covers 8 rows x 64 k = whole 128-byte lines; the 16-byte segments of fragment row b lie
// XOR-swizzled by b / 2 (the lane that fetches segment s of row b sits at position s ^ (b / 2) of the row's eight lanes), so
// that the 16 lanes of a fragment read that hold the same k segment hit 16 different bank groups.  One barrier per stage, behind the
// first two rows of its second half: the wavefronts have read the stage by then, the next one has landed.
// What bounds it at thousands of rows is power: 1280 - 1430 TFLOP/s at a shader clock of 1.8 - 1.9 GHz, where MFMAs alone reach
// 1670 and a large library product 1350.  Two workgroups per CU because a workgroup's start and end (first loads; SwiGLU,
// residual update: 26 bytes per element with seven peers) then run beside the other's MFMAs, and because 128-row tiles leave less of
// the chip idle in the last round.  Against one workgroup of 256 x 256 per CU with both operands through LDS, us:
//   32768 x 14336 x 8192 SwiGLU 5609 -> 5396; 32768 x 8192, residual with 3 peers, K 2048 / 7168 1454 / 3339 -> 1369 / 3249;
//   4001 x 8192, residual with 7 peers, K 1024 / 3584 260 / 345 -> 188 / 277; 2048 x 28672 x 4096 SwiGLU 419 -> 375.
// Whole calls: 8B shape, 2 layers, 2048 rows 1798 -> 1701; 70B R = 8 stage, 4001 rows 3087 -> 2858; R = 4, 32768 rows 12547 -> 12226.
// Columns per wavefront (JT 2, 3, 4) are the cost model's choice: 192 columns where 256 leave half a round idle
// (2048 x 6144 x 4096 106 -> 95 us), 128 for short products.
// Tile order: workgroups are handed to the 8 XCDs round robin by block index and every XCD has its own L2, so block index i is
// mapped to position (i % 8) * (n / 8) + i / 8 of the tile order: each XCD works through one contiguous eighth of it and
// neighbours in the order (which share operands) meet in one L2.  GEMM_GROUP_M row blocks share one column block back to back
// (4 / 6 / 8 / 16: gate/up above 5608 / 5619 / 5396 / 5828 us).
// Rows >= M and weight tiles >= N/16 are clamped on load.  K is a multiple of 64.  Epilogue 0 may split K over workgroups.
// ------------------------------------------------------------------------------------------------
#define DUO_STAGES 3
template <int JT>
__global__ __launch_bounds__(256, 2) void gemm_duo_kernel(GemmArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)   // (buffer descriptors are a device type)
  constexpr int MT = 8, BM = 16 * MT, BN = 64 * JT, S = DUO_STAGES;
  constexpr int XB = BM * 128, XL = BM / 32;   // bytes of a stage, 1 KiB loads per wavefront and stage
  extern __shared__ __attribute__((aligned(16))) unsigned char duo_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = lane & 15, q = lane >> 4;
  const int KT = a.K >> 5, ST = a.K >> 6, NT = a.N >> 4;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const int nblk = gridDim.x, nblk8 = nblk & ~7;   // XCD-aware order
  int bid = (int)blockIdx.x < nblk8 ? ((int)blockIdx.x & 7) * (nblk8 >> 3) + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
  const int ks = bid / (tiles_m * tiles_n);
  bid -= ks * (tiles_m * tiles_n);
  const int per_split = (ST + a.ksplit - 1) / a.ksplit;
  const int s0 = ks * per_split, n = min(ST, s0 + per_split) - s0;   // (the host's plan leaves no split empty)
  const int per_group = GEMM_GROUP_M * tiles_n;
  const int group = bid / per_group, in_group = bid % per_group;
  const int gm = min(GEMM_GROUP_M, tiles_m - group * GEMM_GROUP_M);
  const int m0 = (group * GEMM_GROUP_M + in_group % gm) * BM;
  const int n_blk = in_group / gm;
  const int nt0 = n_blk * (BN / 16) + wave * JT;   // (may lie past the last tile)

  // both operands through buffer descriptors: a uniform base and offset, and 32 bits per lane instead of a 64-bit address per load
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x + (size_t)m0 * a.ldx), 0, -1, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(static_cast<const char*>(a.wp) + (size_t)min(nt0, NT - 1) * KT * 1024), 0, -1, 0x00020000);
  int xsrc[XL], wtile[JT];
#pragma unroll
  for (int i = 0; i < XL; ++i) {   // row group (8 rows) XL wave + i
    const int g = XL * wave + i, r = lane >> 3;
    const int seg = (lane & 7) ^ (((8 * (g & 1) + r) >> 1) & 7);
    xsrc[i] = (min(8 * g + r, a.M - 1 - m0) * a.ldx + seg * 8) * 2;
  }
#pragma unroll
  for (int j = 0; j < JT; ++j) wtile[j] = min(j, max(NT - 1 - nt0, 0)) * KT * 1024;
  // (requests beyond the last stage repeat it: the counts that the waits rely on stay the same to the end)
  auto issue_x = [&](int st, int buf) {
    const int k = (s0 + min(st, n - 1)) * 128;
#pragma unroll
    for (int i = 0; i < XL; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, GEMM2_LDSP(duo_lds + buf * XB + (XL * wave + i) * 1024), 16, xsrc[i], k, 0, 0);
  };
  auto load_w = [&](u32x4_t (&w)[JT], int kt) {
    const int k = (2 * s0 + min(kt, 2 * n - 1)) * 1024;
#pragma unroll
    for (int j = 0; j < JT; ++j) w[j] = __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16, wtile[j] + k, 0);
  };
  f32x4_t acc[JT][MT];
#pragma unroll
  for (int j = 0; j < JT; ++j)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[j][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  // read offsets inside a stage, first and second k tile
  const int xoff0 = (b >> 3) * 1024 + (b & 7) * 128 + ((q) ^ ((b >> 1) & 7)) * 16;
  const int xoff1 = (b >> 3) * 1024 + (b & 7) * 128 + ((4 + q) ^ ((b >> 1) & 7)) * 16;
  u32x4_t w[2][2][JT], f[MT];   // weights [stage parity][k tile], activation fragments of the k tile at hand
  auto row = [&](const u32x4_t (&wk)[JT], int mt) {
#pragma unroll
    for (int j = 0; j < JT; ++j)
      acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wk[j]), __builtin_bit_cast(bf16x8_t, f[mt]), acc[j][mt], 0, 0, 0);
  };
  // Order of a wavefront's requests, stage s: W(s+2, k tile 0) | barrier | X(s+3) | W(s+2, k tile 1); the prologue is what the
  // three stages before the first would have requested.
  // (held in this order: the waits count what was requested behind a stage, and weight loads may otherwise move over the others)
  static_assert(S == 3, "the counts below");
  issue_x(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_w(w[0][0], 0);
  __builtin_amdgcn_sched_barrier(0);
  issue_x(1, 1);
  __builtin_amdgcn_sched_barrier(0);
  load_w(w[0][1], 1);
  __builtin_amdgcn_sched_barrier(0);
  load_w(w[1][0], 2);
  __builtin_amdgcn_sched_barrier(0);
  issue_x(2, 2);
  __builtin_amdgcn_sched_barrier(0);
  load_w(w[1][1], 3);
  ring_meet<2 * XL + 4 * JT>();   // X(0) has landed
  int buf = 0;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) f[mt] = *reinterpret_cast<const u32x4_t*>(duo_lds + xoff0 + mt * 2048);
  auto first_half = [&](const u32x4_t (&wk)[JT]) {   // ... and the fragments of the second
    const unsigned char* const xb = duo_lds + buf * XB + xoff1;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      row(wk, mt);
      f[mt] = *reinterpret_cast<const u32x4_t*>(xb + mt * 2048);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto stage = [&](u32x4_t (&wc)[2][JT], int s) {
    first_half(wc[0]);
    load_w(wc[0], 2 * s + 4);
    __builtin_amdgcn_sched_barrier(0);
    row(wc[1], 0);
    row(wc[1], 1);
    // every wavefront has read the stage (its buffer may be filled again), and X(s+1) has landed: behind it in the queue are
    // W(s, 1), W(s+1, 0), X(s+2), W(s+1, 1), W(s+2, 0)
    ring_meet<XL + 4 * JT>();
    const int next = buf + 1 == S ? 0 : buf + 1;
    const unsigned char* const nx = duo_lds + next * XB + xoff0;
    f[0] = *reinterpret_cast<const u32x4_t*>(nx);
    f[1] = *reinterpret_cast<const u32x4_t*>(nx + 2048);
    issue_x(s + 3, buf);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mt = 2; mt < MT; ++mt) {
      row(wc[1], mt);
      f[mt] = *reinterpret_cast<const u32x4_t*>(nx + mt * 2048);
      __builtin_amdgcn_sched_barrier(0);
    }
    load_w(wc[1], 2 * s + 5);
    __builtin_amdgcn_sched_barrier(0);
    buf = next;
  };
  int s = 0;
  for (; s + 1 < n; s += 2) {
    stage(w[0], s);
    stage(w[1], s + 1);
  }
  if (s < n) {   // (an odd number of stages)
    first_half(w[0][0]);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) row(w[0][1], mt);
  }
  ring_meet<0>();   // the repeated requests land before the LDS is used again or the workgroup ends
  // (the lane is taken afresh from the hardware, so that nothing made from it stays in registers across the loop: three spills less)
  unsigned zero = 0u;
  asm volatile("" : "+v"(zero));
  const int lane_e = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
  if (a.epilogue == 3) {
    gemm_residual_epilogue<MT, JT, 1, 4, 8>(a, acc, duo_lds, m0, n_blk, wave, lane_e);
    return;
  }
  GemmArgs e = a;
  if (a.ksplit > 1) e.out = a.out + (size_t)ks * a.out_stride;
  gemm_epilogue<MT, JT, false>(e, acc, m0, nt0, NT, lane_e);
#endif
}

template <int JT>
static hipError_t launch_gemm_duo(const GemmArgs& a, hipStream_t s) {
  constexpr int RING = DUO_STAGES * 128 * 128, EPI = 64 * GEMM_EPI_STRIDE(64 * JT) * 4;
  static bool prepared[64] = {};
  if ((a.K & 63) || !gemm_duo_reaches(a.ldx, a.K, JT)) return hipErrorInvalidValue;
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(gemm_duo_kernel<JT>), EPI > RING ? EPI : RING, prepared);
  if (e != hipSuccess) return e;
  const int tiles = (a.M + 127) / 128 * ((a.N + 64 * JT - 1) / (64 * JT));
  hipLaunchKernelGGL((gemm_duo_kernel<JT>), dim3(tiles * a.ksplit), dim3(256), a.epilogue == 3 && EPI > RING ? EPI : RING, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Few or ragged rows: BM x BN workgroup tile, WR x WC wavefronts, K in stages of 64 through a ring of S stages in LDS,
// optionally split over ksplit workgroups whose partial products the caller's next kernel adds up.  With up to a few
// hundred rows the product is bound by the one pass over the weights, so what counts is how many bytes of them are in
// flight on how many CUs: S - 1 stages of direct-to-LDS loads per workgroup (80 - 128 KiB, one workgroup per CU) and, by
// the split of K, a workgroup for every CU whatever N is.  Both operands are staged as in gemm_duo_kernel (weights: packed
// tiles as they stand; activations: 8 rows x 64 k per load, XOR-swizzled).  K is a multiple of 32; an odd last k tile
// half-fills its stage.
// Measured (8B shape, us, weights from memory; against 64- or 128-row tiles with register-staged operands and no split):
// 100 rows QKV 68 -> 15.4, O 68 -> 11, gate/up 81 -> 48, down 231 -> 25.5; 64 rows gate/up 84 -> 41.5 (5.7 TB/s), down
// 248 -> 22.8; 2048 rows O 85 -> 63, down 276 -> 205 (1170 TFLOP/s, 128 x 256 tiles).  64 rows x 1280 columns of K 8192: 142 -> 7.3.
// Non-temporal weight loads where one row block covers all rows: gate/up 46.6 -> 41.5 at 64 rows; with several row
// blocks they are 5 - 13 % slower.  A rotated start of the K sweep: no change.
// ------------------------------------------------------------------------------------------------
template <int BM, int BN, int WR, int WC, int S>
__device__ __forceinline__ void gemm_ring_tile(const GemmArgs& a, int block, int nblk) {
  constexpr int WAVES = WR * WC, MT = BM / WR / 16, JT = BN / WC / 16;
  constexpr int XB = BM * 128, WB = BN * 128;             // bytes per stage of 64 k
  constexpr int XL = BM / 8 / WAVES, WL = BN / 8 / WAVES; // 1 KiB loads per wave and stage
  constexpr int L = XL + WL;
  static_assert(XL * WAVES * 8 == BM && WL * WAVES * 8 == BN, "loads divide over the waves");
  extern __shared__ __attribute__((aligned(16))) unsigned char ring_lds[];
  unsigned char* const xring = ring_lds;
  unsigned char* const wring = ring_lds + S * XB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = lane & 15, q = lane >> 4;
  const int wr = wave / WC, wc = wave % WC;
  const int KT = a.K >> 5, ST = (KT + 1) >> 1, NT = a.N >> 4;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const int nblk8 = nblk & ~7;   // XCD-aware order, as in gemm_duo_kernel
  int bid = block < nblk8 ? (block & 7) * (nblk8 >> 3) + (block >> 3) : block;
  const int ks = bid / (tiles_m * tiles_n);
  bid -= ks * (tiles_m * tiles_n);
  const int per_group = GEMM_GROUP_M * tiles_n;
  const int group = bid / per_group, in_group = bid % per_group;
  const int gm = min(GEMM_GROUP_M, tiles_m - group * GEMM_GROUP_M);
  const int m0 = (group * GEMM_GROUP_M + in_group % gm) * BM;
  const int nt0 = in_group / gm * (BN / 16);
  const int per_split = (ST + a.ksplit - 1) / a.ksplit;
  const int s0 = ks * per_split, n = min(ST, s0 + per_split) - s0;   // (the host's plan leaves no split empty)

  const bf16_t* xsrc[XL];
  const u32x4_t* wsrc[WL];
  const int brow = lane >> 3;
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int g = wave + i * WAVES;
    xsrc[i] = a.x + (size_t)min(m0 + 8 * g + brow, a.M - 1) * a.ldx;
  }
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int t = wave + i * WAVES;
    wsrc[i] = reinterpret_cast<const u32x4_t*>(a.wp) + (size_t)min(nt0 + t % (BN / 16), NT - 1) * KT * 64 + lane;
  }
  // one row block: every weight byte is read once and must not push the activations out of the caches (aux 2 = non-temporal)
  const bool once = tiles_m == 1;
  auto issue = [&](int st, int buf) {
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int t = wave + i * WAVES;
      const int kt = min(2 * st + t / (BN / 16), KT - 1);
      if (once) __builtin_amdgcn_global_load_lds(GEMM2_GLBP(wsrc[i] + (size_t)kt * 64), GEMM2_LDSP(wring + buf * WB + t * 1024), 16, 0, 2);
      else __builtin_amdgcn_global_load_lds(GEMM2_GLBP(wsrc[i] + (size_t)kt * 64), GEMM2_LDSP(wring + buf * WB + t * 1024), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int g = wave + i * WAVES;
      const int seg = (lane & 7) ^ (((8 * (g & 1) + brow) >> 1) & 7);
      int k = st * 64 + seg * 8;
      k = k < a.K ? k : k - 32;   // (an odd last k tile: the second half of the stage repeats the first and is not multiplied)
      __builtin_amdgcn_global_load_lds(GEMM2_GLBP(xsrc[i] + k), GEMM2_LDSP(xring + buf * XB + g * 1024), 16, 0, 0);
    }
  };

  f32x4_t acc[JT][MT];
#pragma unroll
  for (int j = 0; j < JT; ++j)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[j][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  const int xrow = (b >> 3) * 1024 + (b & 7) * 128 + wr * (BM / WR) * 128;
  const int xoff0 = xrow + ((q) ^ ((b >> 1) & 7)) * 16, xoff1 = xrow + ((4 + q) ^ ((b >> 1) & 7)) * 16;
  struct Frags { u32x4_t x[MT], w[JT]; };
  auto read = [&](Frags& f, int buf, int h) {
    const unsigned char* xb = xring + buf * XB + (h ? xoff1 : xoff0);
    const unsigned char* wb = wring + buf * WB + h * (BN * 64) + wc * (JT * 1024) + lane * 16;
#pragma unroll
    for (int j = 0; j < JT; ++j) f.w[j] = *reinterpret_cast<const u32x4_t*>(wb + j * 1024);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) f.x[mt] = *reinterpret_cast<const u32x4_t*>(xb + mt * 2048);
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < JT; ++j)
        acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f.w[j]), __builtin_bit_cast(bf16x8_t, f.x[mt]), acc[j][mt], 0, 0, 0);
  };
  // One barrier per stage, between the two halves of its MFMAs.  Before it a wave has its reads of the stage complete
  // and its loads of the next stage landed; behind it the next stage may be read and this stage's buffer be filled.
#pragma unroll
  for (int i = 0; i < S - 1; ++i) issue(s0 + min(i, n - 1), i);
  Frags f0, f1;
  ring_meet<(S - 2) * L>();
  read(f0, 0, 0);
  int buf = 0, fill = S - 1, i = 0;
  for (; i + S - 1 < n; ++i) {
    issue(s0 + i + S - 1, fill);
    read(f1, buf, 1);
    __builtin_amdgcn_sched_barrier(0);
    multiply(f0);
    ring_meet<(S - 2) * L>();
    fill = buf;
    buf = buf + 1 == S ? 0 : buf + 1;
    read(f0, buf, 0);
    __builtin_amdgcn_sched_barrier(0);
    multiply(f1);
    __builtin_amdgcn_sched_barrier(0);
  }
  // the last S - 1 stages: nothing left to request
#pragma unroll
  for (int r = S - 2; r >= 0; --r) {
    if (n - 1 - r >= 0) {
      const bool both = r > 0 || 2 * (s0 + n) <= KT;   // (an odd K / 32: the last stage has one k tile)
      if (both) read(f1, buf, 1);
      __builtin_amdgcn_sched_barrier(0);
      multiply(f0);
      if (r > 0) {
        if (r == S - 2) ring_meet<(S > 2 ? S - 3 : 0) * L>();
        else if (r == S - 3) ring_meet<(S > 3 ? S - 4 : 0) * L>();
        else if (r == S - 4) ring_meet<(S > 4 ? S - 5 : 0) * L>();
        else ring_meet<0>();
        buf = buf + 1 == S ? 0 : buf + 1;
        read(f0, buf, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (both) multiply(f1);
    }
  }
  // with two stages or more, the wait in front of the last one was for everything; a single stage (K <= 64, or a last split of
  // one) leaves the start's other requests, which repeat it, in flight into LDS: they must land before the workgroup ends
  if (n == 1) ring_meet<0>();
  if constexpr (BN == 256 && WR == 2) {   // (whole rows per memory instruction: 8B shape, 2 layers, 1100 rows 1265 -> 1251 us, 2048 1795 -> 1784)
    if (a.epilogue == 3) {
      ring_meet<0>();   // every wavefront is past its last read of the ring, whose memory stages the tile
      gemm_residual_epilogue<MT, JT, WR, WC, 3>(a, acc, ring_lds, m0, nt0 >> 4, wave, lane);
      return;
    }
  }
  GemmArgs e = a;
  if (a.ksplit > 1) e.out = a.out + (size_t)ks * a.out_stride;
  gemm_epilogue<MT, JT, JT == 2>(e, acc, m0 + wr * (BM / WR), nt0 + wc * JT, NT, lane);
}

template <int BM, int BN, int WR, int WC, int S>
__global__ __launch_bounds__(WR * WC * 64) void gemm_ring_kernel(GemmArgs a) {
  gemm_ring_tile<BM, BN, WR, WC, S>(a, (int)blockIdx.x, (int)gridDim.x);
}

// Two products that do not depend on each other in one launch (a's workgroups first): what a short product leaves of the chip at its start and
// end, the other one fills.  The tiles and splits are those that each takes by itself: same bits.
template <int BM_, int BN_, int WR_, int WC_, int S_>
struct RingTile {
  static constexpr int BM = BM_, BN = BN_, WR = WR_, WC = WC_, S = S_, LDS = S_ * (BM_ + BN_) * 128;
  static_assert(WR_ * WC_ == 8, "512 threads");
  static int workgroups(const GemmArgs& g) { return (g.M + BM - 1) / BM * ((g.N + BN - 1) / BN) * g.ksplit; }
};
template <typename A, typename B>
__global__ __launch_bounds__(512) void gemm_ring_pair_kernel(GemmArgs a, GemmArgs b, int n_a) {
  if ((int)blockIdx.x < n_a) gemm_ring_tile<A::BM, A::BN, A::WR, A::WC, A::S>(a, (int)blockIdx.x, n_a);
  else gemm_ring_tile<B::BM, B::BN, B::WR, B::WC, B::S>(b, (int)blockIdx.x - n_a, (int)gridDim.x - n_a);
}
template <typename A, typename B>
static hipError_t launch_ring_pair(const GemmArgs& a, const GemmArgs& b, hipStream_t s) {
  constexpr int LDS = A::LDS > B::LDS ? A::LDS : B::LDS;
  static bool prepared[64] = {};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(gemm_ring_pair_kernel<A, B>), LDS, prepared);
  if (e != hipSuccess) return e;
  const int n_a = A::workgroups(a);
  hipLaunchKernelGGL((gemm_ring_pair_kernel<A, B>), dim3(n_a + B::workgroups(b)), dim3(512), LDS, s, a, b, n_a);
  return hipGetLastError();
}

template <int BM, int BN, int WR, int WC, int S>
static hipError_t launch_gemm_ring_t(const GemmArgs& a, hipStream_t s) {
  constexpr int LDS = S * (BM + BN) * 128;
  static bool prepared[64] = {};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(gemm_ring_kernel<BM, BN, WR, WC, S>), LDS, prepared);
  if (e != hipSuccess) return e;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WR, WC, S>), dim3(tiles_m * tiles_n * a.ksplit), dim3(WR * WC * 64), LDS, s, a);
  return hipGetLastError();
}

static GemmShape shape_of(const GemmArgs& a) { return {a.M, a.N, a.K, a.ldx, a.epilogue, a.n_peers}; }

int gemm_ssq_parts(const GemmArgs& a) {
  // columns per workgroup (256-column tiles) or per wavefront
  static const int cols[TILE_COUNT] = {16, 32, 32, 32, 256, 256, 128, 192, 256};
  const int c = cols[gemm_best_tile(shape_of(a), 1, nullptr)];
  return (a.N + c - 1) / c;
}

int gemm_ksplit(int M, int N, int K, int max_split, float extra_us) { return gemm_best_split(M, N, K, max_split, extra_us); }

// what a product must have, whatever tile it takes (a.ksplit: at least 1 behind it)
static hipError_t check_gemm(GemmArgs& a) {
  if (a.M <= 0 || (a.K & 31) || (a.N & 15) || a.K < 32) return hipErrorInvalidValue;
  if (a.ksplit < 1) a.ksplit = 1;
  if (a.ksplit > 1) {
    const int stages = (a.K + 63) / 64, per = (stages + a.ksplit - 1) / a.ksplit;
    if (a.epilogue != 0 || (stages + per - 1) / per != a.ksplit) return hipErrorInvalidValue;
  }
  // operands of the chosen epilogue
  if (a.epilogue < 0 || a.epilogue > 3) return hipErrorInvalidValue;
  if (a.epilogue == 0 && !a.out) return hipErrorInvalidValue;
  if (a.epilogue == 1 && !a.act) return hipErrorInvalidValue;
  if (a.epilogue == 2 && (!a.q_out || !a.cache_k || !a.cache_v || !a.cos_tab || !a.sin_tab || a.T <= 0 || a.d <= 0)) return hipErrorInvalidValue;
  if (a.epilogue == 3 && (!a.x_res || a.n_peers < 0 || (a.n_peers > 0 && !a.peers) || (a.xh_b && !a.xh_a) || (a.ssq_part && !a.xh_a) ||
                          (a.xh_a && !a.gain_a) || (a.xh_b && !a.gain_b)))
    return hipErrorInvalidValue;
  return hipSuccess;
}

hipError_t launch_gemm_mfma(const GemmArgs& given, hipStream_t s) {
  GemmArgs a = given;
  const hipError_t ok = check_gemm(a);
  if (ok != hipSuccess) return ok;
  const int tile = gemm_best_tile(shape_of(a), a.ksplit, nullptr);
  if (a.epilogue == 3 && (tile == TILE_64x64 || (tile == TILE_256x256 && a.n_peers > 0))) return hipErrorInvalidValue;   // (their kernels do not have it)
  switch (tile) {
    case TILE_64x64: return launch_gemm_ring_t<64, 64, 2, 4, 6>(a, s);
    case TILE_64x128: return launch_gemm_ring_t<64, 128, 2, 4, 6>(a, s);
    case TILE_128x64: return launch_gemm_ring_t<128, 64, 4, 2, 5>(a, s);
    case TILE_128x128: return launch_gemm_ring_t<128, 128, 2, 4, 5>(a, s);
    case TILE_128x256: return launch_gemm_ring_t<128, 256, 2, 4, 3>(a, s);
    case TILE_256x256: return launch_gemm_lds(a, s);
    case TILE_DUO_128: return launch_gemm_duo<2>(a, s);
    case TILE_DUO_192: return launch_gemm_duo<3>(a, s);
    default: return launch_gemm_duo<4>(a, s);
  }
}

// The pairs of tiles that two products of up to 128 rows take (and most of up to 256), the second one's tile the larger: its workgroups take longest, so
// they go first
static int pair_of(const GemmArgs& a, const GemmArgs& b, bool* swap) {
  if (a.epilogue == 3 || b.epilogue == 3) return -1;
  int ta = gemm_best_tile(shape_of(a), std::max(1, a.ksplit), nullptr), tb = gemm_best_tile(shape_of(b), std::max(1, b.ksplit), nullptr);
  const auto rank = [](int t) { return t == TILE_64x64 ? 0 : t == TILE_128x64 ? 1 : t == TILE_128x128 ? 2 : -1; };
  ta = rank(ta);
  tb = rank(tb);
  if (ta < 0 || tb < 0) return -1;
  *swap = ta > tb;
  return *swap ? tb * 3 + ta : ta * 3 + tb;
}
bool gemm_pairs(const GemmArgs& a, const GemmArgs& b) {
  bool swap;
  return pair_of(a, b, &swap) >= 0;
}
hipError_t launch_gemm_pair(const GemmArgs& given_a, const GemmArgs& given_b, hipStream_t s) {
  GemmArgs a = given_a, b = given_b;
  hipError_t e = check_gemm(a);
  if (e == hipSuccess) e = check_gemm(b);
  if (e != hipSuccess) return e;
  bool swap = false;
  const int pair = pair_of(a, b, &swap);
  if (swap) std::swap(a, b);
  typedef RingTile<64, 64, 2, 4, 6> Small;
  typedef RingTile<128, 64, 4, 2, 5> Tall;
  typedef RingTile<128, 128, 2, 4, 5> Large;
  switch (pair) {
    case 0: return launch_ring_pair<Small, Small>(a, b, s);
    case 1: return launch_ring_pair<Tall, Small>(b, a, s);
    case 2: return launch_ring_pair<Large, Small>(b, a, s);
    case 4: return launch_ring_pair<Tall, Tall>(a, b, s);
    case 5: return launch_ring_pair<Large, Tall>(b, a, s);
    case 8: return launch_ring_pair<Large, Large>(a, b, s);
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------------------------------------
// Causal GQA flash attention for T new tokens per sequence over the cache (which already holds
// them).  Everything is computed transposed so that no operand needs a shuffle:
//   S^T[key][query] = K Q^T       A = K tile (16 keys x 32 dims, straight from the row-major K cache),
//                                 B = Q^T (16 queries x 32 dims, kept in registers);
//   a lane then owns, for ITS query (lane%16), keys 4*(lane/16)+r of each 16-key tile: the softmax
//   statistics of a query need two shuffles, and the lane's 8 probabilities of a 32-key block are,
//   as they stand, the B operand of
//   O^T[dim][query] = V^T P^T     A = V^T tile (16 dims x 32 keys) from the transposed V cache, with
//                                 the same key order (two 8-byte loads per lane).
// One wavefront owns QT tiles of 16 queries of one q head; a workgroup = 4 wavefronts.
// ------------------------------------------------------------------------------------------------
template <int D, int QT>
__global__ __launch_bounds__(256) void attn_prefill_kernel(AttnPrefillArgs a) {
  constexpr int DS = D / 32;  // 32-dim slabs
  constexpr int DT = D / 16;  // 16-dim output tiles
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int b = lane & 15, q = lane >> 4;
  const int n_qblk = gridDim.x;
  const int qblk = n_qblk - 1 - blockIdx.x;  // longest rows first
  const int h = blockIdx.y, bi = blockIdx.z;
  const int kvh = h / (a.nq / a.nkv);
  const int t0 = (qblk * 4 + wave) * QT * 16;
  if (t0 >= a.T) return;
  const float scale = 1.0f / sqrtf((float)D);
  const uint4 zero4 = make_uint4(0, 0, 0, 0);

  uint4 qreg[QT][DS];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int t = t0 + qt * 16 + b;
#pragma unroll
    for (int s = 0; s < DS; ++s)
      qreg[qt][s] = t < a.T ? *reinterpret_cast<const uint4*>(a.q + ((size_t)bi * a.T + t) * a.nq * D + h * D +
                                                              s * 32 + q * 8)
                            : zero4;
  }
  f32x4_t oacc[QT][DT];
  float mrun[QT], lrun[QT];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    mrun[qt] = -INFINITY;
    lrun[qt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[qt][dt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  }
  const bf16_t* kc = a.cache_k + ((size_t)bi * a.nkv + kvh) * a.max_seq * D;
  const bf16_t* vc = a.cache_v + ((size_t)bi * a.nkv + kvh) * D * a.max_seq;
  const int last_t = min(a.T, t0 + QT * 16) - 1;
  const int n_keys = a.pos0 + last_t + 1;

  for (int kb = 0; kb < n_keys; kb += 32) {
    uint4 kreg[2][DS];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int s = 0; s < DS; ++s)
        kreg[t][s] = *reinterpret_cast<const uint4*>(kc + (size_t)(kb + 16 * t + b) * D + s * 32 + q * 8);
    uint4 vreg[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16_t* vp = vc + (size_t)(dt * 16 + b) * a.max_seq + kb + 4 * q;
      const uint2 lo = *reinterpret_cast<const uint2*>(vp);
      const uint2 hi = *reinterpret_cast<const uint2*>(vp + 16);
      vreg[dt] = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      f32x4_t st[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        st[t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < DS; ++s) st[t] = mfma16(kreg[t][s], qreg[qt][s], st[t]);
      }
      const int qpos = a.pos0 + t0 + qt * 16 + b;
      float sv[8];
      float mloc = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = kb + 16 * t + 4 * q + r;
          const float v = key <= qpos ? st[t][r] * scale : -INFINITY;
          sv[t * 4 + r] = v;
          mloc = fmaxf(mloc, v);
        }
      mloc = fmaxf(mloc, __shfl_xor(mloc, 16, 64));
      mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
      const float mnew = fmaxf(mrun[qt], mloc);   // finite from the first block on (key 0 is always visible)
      const float corr = __expf(mrun[qt] - mnew);
      float psum = 0.f;
      float pv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pv[e] = __expf(sv[e] - mnew);
        psum += pv[e];
      }
      lrun[qt] = lrun[qt] * corr + psum;
      mrun[qt] = mnew;
      uint4 pb;
      pb.x = f32_to_bf16x2(pv[0], pv[1]);
      pb.y = f32_to_bf16x2(pv[2], pv[3]);
      pb.z = f32_to_bf16x2(pv[4], pv[5]);
      pb.w = f32_to_bf16x2(pv[6], pv[7]);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) oacc[qt][dt][r] *= corr;
        oacc[qt][dt] = mfma16(vreg[dt], pb, oacc[qt][dt]);
      }
    }
  }
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    float l = lrun[qt];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    const float inv = 1.0f / l;
    const int t = t0 + qt * 16 + b;
    if (t < a.T) {
      bf16_t* op = a.o + ((size_t)bi * a.T + t) * a.nq * D + h * D;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        uint2 pk;
        pk.x = f32_to_bf16x2(oacc[qt][dt][0] * inv, oacc[qt][dt][1] * inv);
        pk.y = f32_to_bf16x2(oacc[qt][dt][2] * inv, oacc[qt][dt][3] * inv);
        *reinterpret_cast<uint2*>(op + dt * 16 + 4 * q) = pk;
      }
    }
  }
}

// the largest of the four lanes that hold one query, 16, 32 and 48 lanes apart, by exchanging rows of 16 and halves
__device__ __forceinline__ float max_over_rows(float v) {
  typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2_t;
  u32x2_t r = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// ------------------------------------------------------------------------------------------------
// The same computation with the K / V^T tiles of a 32-key block staged once per workgroup in LDS
// (double buffered) and shared by its 4 wavefronts, each of which owns QT tiles of 16 queries of
// one q head.  With grouped-query attention the wavefronts of a workgroup are HW = min(G, 4) q heads
// of ONE kv head over the same query block, so they walk exactly the same keys.
// What bounds it is the vector work of the softmax between the matrix instructions (a tile of 16 queries x 32 keys is 16
// of those and eight probabilities per lane), so that is kept short: scores stay unscaled and scale and base-2 exponent
// are one fused multiply-add; keys are masked only in the blocks that cross the diagonal; the maximum travels by row swaps
// instead of through LDS; and the output is rescaled only where a maximum of the tile has grown.  (Letting it grow by 2^6
// before rescaling would save another 0.5 % of a call, but the largest weight of a query is then no longer exactly 1 and its
// bf16 rounding shows: attention output behind 4001 positions 1.297e-2 -> 1.312e-2 of its norm.)  The K rows are staged in the order that leaves a
// lane eight neighbouring keys (row 16 t + i holds key 8 (i / 4) + 4 t + i % 4), so its share of V^T is one 16-byte read.
// us per layer (direct kernel -> now): 16 x 2048 tokens, 16 q / 2 kv heads 556 -> 389 (710 TFLOP/s); 1 x 2048, 32 / 8 heads 156 -> 73;
// 1 x 4001, 8 / 1 heads 202 -> 93; 1 x 100, 32 / 8 heads 12.8 -> 6.0.
// ------------------------------------------------------------------------------------------------
template <int D, int HW, int QT>
__global__ __launch_bounds__(256, 2) void attn_prefill_lds_kernel(AttnPrefillArgs a, int n_pairs) {
  constexpr int DS = D / 32, DT = D / 16;
  constexpr int QW = 4 / HW;                 // query sub-blocks (of QT * 16) per workgroup
  constexpr int KROW = D * 2 + 16;           // bytes per staged K row (key): 16-byte pad, conflict-free b128 reads
  constexpr int VROW = 64 + 16;              // bytes per staged V^T row (dim): 32 keys + pad
  constexpr int KBYTES = 32 * KROW, VBYTES = D * VROW;
  constexpr int SEGS = D / 64;               // 16-byte segments per thread and tile
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][KBYTES + VBYTES];

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int b = lane & 15, q = lane >> 4;
  // Workgroups are dispatched in block order, one to each of 256 CUs, then a second one and so on, and a causal one is as long as its
  // queries are far back.  So: longest first over all (sequence, head group) pairs, and where all of them fit the chip at once (one query tile) every
  // second row of 256 in reverse, so that the sum on each CU is about the same.  (Pairs vary fastest: the workgroups of one pair share an XCD's L2
  // where the pairs are a multiple of 8.)
  const int n_wg = (int)gridDim.x, id = (int)blockIdx.x, row = id >> 8;
  const int rank = QT == 1 && (row & 1) ? (row << 8) + min(256, n_wg - (row << 8)) - 1 - (id & 255) : id;
  const int pair = rank % n_pairs, hg = pair % (a.nq / HW), bi = pair / (a.nq / HW);
  const int qblk = n_wg / n_pairs - 1 - rank / n_pairs;
  const int h = hg * HW + wave % HW;
  const int kvh = h / (a.nq / a.nkv);
  const int t0 = (qblk * QW + wave / HW) * (QT * 16);       // this wavefront's first query
  const float scale2 = 1.4426950408889634f / sqrtf((float)D);   // scores to exponents of 2

  uint4 qreg[QT][DS];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int t = min(t0 + qt * 16 + b, a.T - 1);           // rows past T: a valid address, never stored
#pragma unroll
    for (int s = 0; s < DS; ++s)
      qreg[qt][s] = *reinterpret_cast<const uint4*>(a.q + ((size_t)bi * a.T + t) * a.nq * D + h * D + s * 32 + q * 8);
  }
  f32x4_t oacc[QT][DT];
  float mrun[QT], lrun[QT];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    mrun[qt] = -INFINITY;
    lrun[qt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[qt][dt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  }
  const bf16_t* kc = a.cache_k + ((size_t)bi * a.nkv + kvh) * a.max_seq * D;
  const bf16_t* vc = a.cache_v + ((size_t)bi * a.nkv + kvh) * D * a.max_seq;
  const int wg_last_t = min(a.T, (qblk + 1) * QW * QT * 16) - 1;
  const int n_keys = a.pos0 + wg_last_t + 1;                 // keys the workgroup walks (same for all its waves)
  const int my_last = a.pos0 + min(a.T - 1, t0 + QT * 16 - 1);  // last position this wavefront's queries see
  const int n_blk = (n_keys + 31) / 32;

  u32x4_t kst[SEGS], vst[SEGS];
  auto fetch = [&](int blk) {   // global -> registers (unconditional: blk is clamped by the caller)
    const int kb = blk * 32;
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
      const int seg = tid + 256 * i;
      const int krow = seg / (D / 8), kcx = seg % (D / 8);
      kst[i] = *reinterpret_cast<const u32x4_t*>(kc + (size_t)(kb + krow) * D + kcx * 8);
      const int vrow = seg >> 2, vcx = seg & 3;
      vst[i] = *reinterpret_cast<const u32x4_t*>(vc + (size_t)vrow * a.max_seq + kb + vcx * 8);
    }
  };
  auto stash = [&](int buf) {   // registers -> LDS
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
      const int seg = tid + 256 * i;
      const int key = seg / (D / 8), kcx = seg % (D / 8);
      const int krow = 16 * ((key >> 2) & 1) + 4 * (key >> 3) + (key & 3);
      *reinterpret_cast<u32x4_t*>(&lds[buf][krow * KROW + kcx * 16]) = kst[i];
      const int vrow = seg >> 2, vcx = seg & 3;
      *reinterpret_cast<u32x4_t*>(&lds[buf][KBYTES + vrow * VROW + vcx * 16]) = vst[i];
    }
  };

  fetch(0);
  stash(0);
  __syncthreads();
  for (int blk = 0; blk < n_blk; ++blk) {
    const int buf = blk & 1;
    const int kb = blk * 32;
    fetch(min(blk + 1, n_blk - 1));   // next block's tiles travel while this one is computed
    if (kb <= my_last && t0 < a.T) {
      const unsigned char* kl = &lds[buf][0];
      const unsigned char* vl = &lds[buf][KBYTES];
      f32x4_t st[QT][2];
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) st[qt][0] = st[qt][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < DS; ++s) {
          const uint4 kf = *reinterpret_cast<const uint4*>(kl + (16 * t + b) * KROW + s * 64 + q * 16);
#pragma unroll
          for (int qt = 0; qt < QT; ++qt) st[qt][t] = mfma16(kf, qreg[qt][s], st[qt][t]);
        }
      uint4 pb[QT];
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        // st[t][r] is the score of this lane's query with key kb + 8 q + 4 t + r
        if (kb + 31 > a.pos0 + t0 + qt * 16) {   // (uniform) the block crosses the diagonal of the tile
          const int visible = a.pos0 + t0 + qt * 16 + b - kb - 8 * q;   // the lane's keys 0 .. visible are
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) st[qt][t][r] = 4 * t + r <= visible ? st[qt][t][r] : -INFINITY;
        }
        float mloc = fmaxf(fmaxf(fmaxf(st[qt][0][0], st[qt][0][1]), fmaxf(st[qt][0][2], st[qt][0][3])),
                           fmaxf(fmaxf(st[qt][1][0], st[qt][1][1]), fmaxf(st[qt][1][2], st[qt][1][3])));
        mloc = max_over_rows(mloc);   // (finite in the first block: key 0 is always visible)
        if (__any(mloc > mrun[qt])) {   // uniform; the first block always
          const float mnew = fmaxf(mrun[qt], mloc);
          const float corr = __builtin_amdgcn_exp2f((mrun[qt] - mnew) * scale2);
          lrun[qt] *= corr;
          mrun[qt] = mnew;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 4; ++r) oacc[qt][dt][r] *= corr;
        }
        const float base = -mrun[qt] * scale2;
        float pv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(fmaf(st[qt][e >> 2][e & 3], scale2, base));
        lrun[qt] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
        pb[qt].x = f32_to_bf16x2(pv[0], pv[1]);
        pb[qt].y = f32_to_bf16x2(pv[2], pv[3]);
        pb[qt].z = f32_to_bf16x2(pv[4], pv[5]);
        pb[qt].w = f32_to_bf16x2(pv[6], pv[7]);
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint4 vf = *reinterpret_cast<const uint4*>(vl + (dt * 16 + b) * VROW + q * 16);
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) oacc[qt][dt] = mfma16(vf, pb[qt], oacc[qt][dt]);
      }
    }
    stash(buf ^ 1);   // that buffer was last read before the previous barrier
    __syncthreads();
  }
  if (t0 >= a.T) return;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    float l = lrun[qt];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    const float inv = 1.0f / l;
    const int t = t0 + qt * 16 + b;
    if (t < a.T) {
      bf16_t* op = a.o + ((size_t)bi * a.T + t) * a.nq * D + h * D;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        uint2 pk;
        pk.x = f32_to_bf16x2(oacc[qt][dt][0] * inv, oacc[qt][dt][1] * inv);
        pk.y = f32_to_bf16x2(oacc[qt][dt][2] * inv, oacc[qt][dt][3] * inv);
        *reinterpret_cast<uint2*>(op + dt * 16 + 4 * q) = pk;
      }
    }
  }
}

template <int D, int QT>
static hipError_t launch_attn_prefill_lds(const AttnPrefillArgs& a, int hw, int n_wg, int n_pairs, hipStream_t s) {
  const dim3 grid(n_wg), block(256);
  if (hw == 4) hipLaunchKernelGGL((attn_prefill_lds_kernel<D, 4, QT>), grid, block, 0, s, a, n_pairs);
  else if (hw == 2) hipLaunchKernelGGL((attn_prefill_lds_kernel<D, 2, QT>), grid, block, 0, s, a, n_pairs);
  else hipLaunchKernelGGL((attn_prefill_lds_kernel<D, 1, QT>), grid, block, 0, s, a, n_pairs);
  return hipGetLastError();
}

// 16-query tiles per wavefront: one, of which four workgroups are resident per CU, until they are more than a quarter beyond what the chip holds
// (then the last ones run on a nearly empty chip); else two, which read K / V^T from LDS half as often (three: 5 - 14 % slower than two everywhere).
// us, one / two tiles: 8B shape 1 x 1000 31 / 43, 1 x 2048 (1024 workgroups of one tile) 73 / 83, 1 x 2600 (1304) 104 / 109, 3 x 1000 (1512) 61 / 53, 1 x 8000
// 837 / 658; 70B R = 8 1 x 4001 93 / 137, 2 x 5000 (1252) 186 / 208; R = 4 1 x 5000 (1252) 182 / 207, 1 x 6000 (1500) 281 / 255, 16 x 2048 481 / 389.
// Longest first within each pair only, and one to three tiles by which fit twice per CU: 8B 1 x 2048 123, 4 x 1000 99 (61), R = 8 1 x 4001 126, R = 4 16 x 2048 460.
#define ATTN_ONE_TILE_WORKGROUPS 1280
template <int D>
static hipError_t launch_attn_prefill_lds(const AttnPrefillArgs& a, hipStream_t s) {
  const int g = a.nq / a.nkv;
  const int hw = g >= 4 && g % 4 == 0 ? 4 : (g % 2 == 0 ? 2 : 1);
  const int n_pairs = a.nq / hw * a.B;
  const auto workgroups = [&](int qt) { return (long long)((a.T + 64 / hw * qt - 1) / (64 / hw * qt)) * n_pairs; };
  if (workgroups(2) > 0x7fffffffll) return hipErrorInvalidValue;
  if (workgroups(1) <= ATTN_ONE_TILE_WORKGROUPS) return launch_attn_prefill_lds<D, 1>(a, hw, (int)workgroups(1), n_pairs, s);
  return launch_attn_prefill_lds<D, 2>(a, hw, (int)workgroups(2), n_pairs, s);
}

hipError_t launch_attn_prefill(const AttnPrefillArgs& a, hipStream_t s) {
  // the LDS-shared kernel (its reads run to the end of the last 32-key block, which the cache capacity, a multiple of 128,
  // always covers); the direct one where a prompt is two key blocks at most and the staging costs more than it saves
  // (8B shape, one layer, us, direct / shared: 60 tokens 123 / 129, 8 x 60 268 / 270, 100 132 / 125, 200 191 / 181)
  if (a.T > 64 && (a.max_seq & 31) == 0) {
    if (a.d == 128) return launch_attn_prefill_lds<128>(a, s);
    if (a.d == 64) return launch_attn_prefill_lds<64>(a, s);
    return hipErrorInvalidValue;
  }
  constexpr int QT = 2;
  const int bq = 4 * QT * 16;
  const dim3 grid((a.T + bq - 1) / bq, a.nq, a.B);
  if (a.d == 128) hipLaunchKernelGGL((attn_prefill_kernel<128, QT>), grid, dim3(256), 0, s, a);
  else if (a.d == 64) hipLaunchKernelGGL((attn_prefill_kernel<64, QT>), grid, dim3(256), 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
