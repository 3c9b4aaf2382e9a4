// Plain kernels: any size, both storage types, fp32 arithmetic.  They are the whole path for the
// fp32 storage type and the fallback of the bf16 one; reduce_norm is used by both paths, rope_append and
// swiglu_parts by the streaming / MFMA path.  gfx950 only.
#include "common.h"

// ------------------------------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ void load4(const T* p, float v[4]);
template <> __device__ __forceinline__ void load4<float>(const float* p, float v[4]) {
  float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
template <> __device__ __forceinline__ void load4<bf16_t>(const bf16_t* p, float v[4]) {
  uint2 t = *reinterpret_cast<const uint2*>(p);
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xFFFF0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xFFFF0000u);
}
template <typename T> __device__ __forceinline__ void store4(T* p, const float v[4]);
template <> __device__ __forceinline__ void store4<float>(float* p, const float v[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t* p, const float v[4]) {
  uint2 t;
  t.x = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
  t.y = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
  *reinterpret_cast<uint2*>(p) = t;
}

// ------------------------------------------------------------------------------------------------
// Reduce + residual add + RMSNorm: the local image of the residual update and the norm that follows it
// (Algorithm 1) with the AllReduce written as a sum over rank partial sums (Eq. 2).
// One workgroup per row; the summation order is fixed: x, parts 0.., peers 0.. .
// ------------------------------------------------------------------------------------------------
// The squares of four columns, in an order that is written out: left to the compiler, two kernels around it may round differently, and the schedules
// that call for one or the other are to give the same bits.
__device__ __forceinline__ float squares4(const float (&v)[4]) { return fmaf(v[3], v[3], fmaf(v[2], v[2], fmaf(v[0], v[0], v[1] * v[1]))); }

// f(s, N) for the pieces 0 .. n - 1 of a sum, four at a time: what N pieces read is requested before the first of them is added, in order.  One by one each was
// a round trip to memory of its own (other XCDs have just written them), for each of up to eight partial products and seven peers.  With rotary + append and SwiGLU
// in one launch where modules share launches, us, before / after: 1.2B (4 layers) prompt of 60 167 / 161, 20 sequences behind 200 positions, 8 steps 1695 / 1652; 70B R = 8 (2)
// 40 behind 700 1465 / 1412, 900 rows 600 / 593; R = 4 (2) 230 rows 371 / 366; 1.2B (8) 3 x 333 and 8 steps 2959 / 2930; 8B (2) batch 64 2871 / 2866.
template <int N> struct Pieces { static constexpr int n = N; };
template <typename F>
__device__ __forceinline__ void four_at_a_time(int n, const F& f) {
  int s = 0;
  for (; s + 4 <= n; s += 4) f(s, Pieces<4>());
  if (n - s == 3) f(s, Pieces<3>());
  else if (n - s == 2) f(s, Pieces<2>());
  else if (n - s == 1) f(s, Pieces<1>());
}

// x += the partial sums and peers of r, for the columns col[] of the row that starts at element `row`
template <typename T, int C>
__device__ __forceinline__ void reduce_add(const ReduceNormArgs& r, size_t row, const int (&col)[C], float (&x)[C][4]) {
  auto add = [&](int n, auto load) {
    four_at_a_time(n, [&](int s, auto pieces) {
      constexpr int N = decltype(pieces)::n;
      float t[N][C][4];
#pragma unroll
      for (int j = 0; j < N; ++j)
#pragma unroll
        for (int c = 0; c < C; ++c) load(s + j, row + col[c], t[j][c]);
#pragma unroll
      for (int j = 0; j < N; ++j)
#pragma unroll
        for (int c = 0; c < C; ++c)
          for (int e = 0; e < 4; ++e) x[c][e] += t[j][c][e];
    });
  };
  add(r.n_parts, [&](int s, size_t at, float (&t)[4]) { load4<float>(r.parts + s * r.part_stride + at, t); });
  add(r.n_peers, [&](int s, size_t at, float (&t)[4]) { load4<T>(reinterpret_cast<const T*>(r.peers) + s * r.peer_stride + at, t); });
}

// STEP: x_out takes the step (a.x_step), for which the old values stay in registers past the sums; a branch of one kernel cost every
// reduce of a wide decode step 0.2 - 0.3 us (1.2B, 4 layers, 50 sequences, 8 steps 2692 -> 2675 us).
// The row stays in registers (C pieces of 4 columns per thread), and the gains are requested before the sums of squares meet.
template <typename T, bool STEP, int C>
__global__ __launch_bounds__(1024) void reduce_norm_kernel(ReduceNormArgs a) {
  const int H = a.H, step = blockDim.x * 4;
  const size_t row = (size_t)blockIdx.x * H;
  const T* const emb = reinterpret_cast<const T*>(a.emb);
  const float* const src = a.x_src ? a.x_src : a.x;
  int col[C];   // (columns behind the row's end: its last ones again, not stored)
  float v[C][4], old[C][4], g[2][C][4], ss = 0.f;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    col[c] = min((int)threadIdx.x * 4 + c * step, H - 4);
    if (emb) load4<T>(emb + row + col[c], v[c]);
    else load4<float>(src + row + col[c], v[c]);
    for (int e = 0; e < 4; ++e) old[c][e] = v[c][e];
  }
  reduce_add<T>(a, row, col, v);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    if ((int)threadIdx.x * 4 + c * step >= H) break;
    store4<float>(a.x + row + col[c], v[c]);
    if (STEP) {
      float t[4];
      for (int e = 0; e < 4; ++e) t[e] = v[c][e] - old[c][e];
      store4<float>(a.x_out + row + col[c], t);
    } else if (a.x_out) {
      store4<float>(a.x_out + row + col[c], v[c]);
    }
    ss += squares4(v[c]);
  }
  if (!a.out_a && !a.out_b) return;
  auto gains = [&](const void* gain, float (&to)[C][4]) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if (gain) load4<T>(reinterpret_cast<const T*>(gain) + col[c], to[c]);
      else to[c][0] = to[c][1] = to[c][2] = to[c][3] = 1.f;
    }
  };
  if (a.out_a) gains(a.gain_a, g[0]);
  if (a.out_b) gains(a.gain_b, g[1]);
  __shared__ float red[16];
  ss = wave_sum(ss);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  if (lane == 0) red[wave] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < nw; ++w) tot += red[w];
  const float rs = 1.0f / sqrtf(tot / (float)H + a.eps);
  auto give = [&](void* out, const float (&by)[C][4]) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if ((int)threadIdx.x * 4 + c * step >= H) break;
      float y[4];
      for (int e = 0; e < 4; ++e) y[e] = v[c][e] * rs * by[c][e];
      store4<T>(reinterpret_cast<T*>(out) + row + col[c], y);
    }
  };
  if (a.out_a) give(a.out_a, g[0]);
  if (a.out_b) give(a.out_b, g[1]);
}

// ... rows that are too long for that
template <typename T, bool STEP>
__global__ void reduce_norm_long_kernel(ReduceNormArgs a) {
  const int row = blockIdx.x;
  const int H = a.H;
  float* xr = a.x + (size_t)row * H;
  const T* emb = reinterpret_cast<const T*>(a.emb);
  const T* peers = reinterpret_cast<const T*>(a.peers);
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < H; i += blockDim.x * 4) {
    float v[4], t[4];
    if (emb) load4<T>(emb + (size_t)row * H + i, v);
    else load4<float>(a.x_src ? a.x_src + (size_t)row * H + i : xr + i, v);
    const float old[4] = {v[0], v[1], v[2], v[3]};
    for (int s = 0; s < a.n_parts; ++s) {
      load4<float>(a.parts + s * a.part_stride + (size_t)row * H + i, t);
      v[0] += t[0]; v[1] += t[1]; v[2] += t[2]; v[3] += t[3];
    }
    for (int j = 0; j < a.n_peers; ++j) {
      load4<T>(peers + j * a.peer_stride + (size_t)row * H + i, t);
      v[0] += t[0]; v[1] += t[1]; v[2] += t[2]; v[3] += t[3];
    }
    store4<float>(xr + i, v);
    if (STEP) {
      for (int e = 0; e < 4; ++e) t[e] = v[e] - old[e];
      store4<float>(a.x_out + (size_t)row * H + i, t);
    } else if (a.x_out) {
      store4<float>(a.x_out + (size_t)row * H + i, v);
    }
    ss += squares4(v);
  }
  if (!a.out_a && !a.out_b) return;
  __shared__ float red[16];
  ss = wave_sum(ss);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  if (lane == 0) red[wave] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < nw; ++w) tot += red[w];
  const float rs = 1.0f / sqrtf(tot / (float)H + a.eps);
  T* oa = reinterpret_cast<T*>(a.out_a);
  T* ob = reinterpret_cast<T*>(a.out_b);
  const T* ga = reinterpret_cast<const T*>(a.gain_a);
  const T* gb = reinterpret_cast<const T*>(a.gain_b);
  for (int i = threadIdx.x * 4; i < H; i += blockDim.x * 4) {
    float v[4], g[4], y[4];
    load4<float>(xr + i, v);  // this thread's own writes
    if (oa) {
      if (ga) load4<T>(ga + i, g);
      else g[0] = g[1] = g[2] = g[3] = 1.f;
      for (int e = 0; e < 4; ++e) y[e] = v[e] * rs * g[e];
      store4<T>(oa + (size_t)row * H + i, y);
    }
    if (ob) {
      if (gb) load4<T>(gb + i, g);
      else g[0] = g[1] = g[2] = g[3] = 1.f;
      for (int e = 0; e < 4; ++e) y[e] = v[e] * rs * g[e];
      store4<T>(ob + (size_t)row * H + i, y);
    }
  }
}

template <typename T, bool STEP>
static void launch_reduce_norm_t(const ReduceNormArgs& a, int threads, hipStream_t s) {
  auto* const kernel = a.H <= 4 * threads ? reduce_norm_kernel<T, STEP, 1> : a.H <= 8 * threads ? reduce_norm_kernel<T, STEP, 2>
                       : a.H <= 16 * threads ? reduce_norm_kernel<T, STEP, 4> : reduce_norm_long_kernel<T, STEP>;
  hipLaunchKernelGGL(kernel, dim3(a.rows), dim3(threads), 0, s, a);
}
hipError_t launch_reduce_norm(const ReduceNormArgs& a, bool is_bf16, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  const int threads = a.H >= 4096 ? 1024 : 256;
  const bool step = a.x_out && a.x_step;
  if (is_bf16) step ? launch_reduce_norm_t<bf16_t, true>(a, threads, s) : launch_reduce_norm_t<bf16_t, false>(a, threads, s);
  else step ? launch_reduce_norm_t<float, true>(a, threads, s) : launch_reduce_norm_t<float, false>(a, threads, s);
  return hipGetLastError();
}

// Two reduces of a stream in one pass (modules m and m + 1, whose outputs are both there): a's partial sums and peers, whose rows a's outputs are made
// from, then b's; the rows stay in registers (C pieces of 4 columns per thread) and only the second ones are stored.  Same order of sums as one by one.
template <typename T, int C>
__global__ __launch_bounds__(1024) void reduce_norm_two_kernel(ReduceNormArgs a, ReduceNormArgs b) {
  const int H = a.H, step = blockDim.x * 4;
  const size_t row = (size_t)blockIdx.x * H;
  __shared__ float red[2][16];
  int col[C];
  float v[2][C][4], ss[2] = {0.f, 0.f};
#pragma unroll
  for (int c = 0; c < C; ++c) {
    col[c] = min((int)threadIdx.x * 4 + c * step, H - 4);
    load4<float>(a.x + row + col[c], v[0][c]);
  }
  reduce_add<T>(a, row, col, v[0]);
#pragma unroll
  for (int c = 0; c < C; ++c)
    for (int e = 0; e < 4; ++e) v[1][c][e] = v[0][c][e];
  reduce_add<T>(b, row, col, v[1]);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    if ((int)threadIdx.x * 4 + c * step >= H) break;
    ss[0] += squares4(v[0][c]);
    ss[1] += squares4(v[1][c]);
    store4<float>(b.x + row + col[c], v[1][c]);
    if (b.x_out) store4<float>(b.x_out + row + col[c], v[1][c]);
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    ss[k] = wave_sum(ss[k]);
    if (lane == 0) red[k][wave] = ss[k];
  }
  __syncthreads();
  auto give = [&](const float (&w)[C][4], const float* sums, void* out, const void* gain) {
    if (!out) return;
    float tot = 0.f;
    for (int k = 0; k < nw; ++k) tot += sums[k];
    const float rs = 1.0f / sqrtf(tot / (float)H + a.eps);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int i = threadIdx.x * 4 + c * step;
      if (i >= H) break;
      float g[4] = {1.f, 1.f, 1.f, 1.f}, y[4];
      if (gain) load4<T>(reinterpret_cast<const T*>(gain) + i, g);
      for (int e = 0; e < 4; ++e) y[e] = w[c][e] * rs * g[e];
      store4<T>(reinterpret_cast<T*>(out) + row + i, y);
    }
  };
  give(v[0], red[0], a.out_a, a.gain_a);
  give(v[0], red[0], a.out_b, a.gain_b);
  give(v[1], red[1], b.out_a, b.gain_a);
  give(v[1], red[1], b.out_b, b.gain_b);
}

// (the threads per row of launch_reduce_norm: the same sums)
bool reduce_norm_two_fits(int H) { return H % 4 == 0 && H <= 2 * 4 * (H >= 4096 ? 1024 : 256) * (H >= 4096 ? 1 : 2); }
hipError_t launch_reduce_norm_two(const ReduceNormArgs& a, const ReduceNormArgs& b, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  if (!reduce_norm_two_fits(a.H) || a.H != b.H || a.rows != b.rows || a.x != b.x || a.emb || b.emb || a.x_src || b.x_src || a.x_out || b.x_step) return hipErrorInvalidValue;
  const int threads = a.H >= 4096 ? 1024 : 256;
  if (a.H <= 4 * threads) hipLaunchKernelGGL((reduce_norm_two_kernel<bf16_t, 1>), dim3(a.rows), dim3(threads), 0, s, a, b);
  else if (a.H <= 8 * threads) hipLaunchKernelGGL((reduce_norm_two_kernel<bf16_t, 2>), dim3(a.rows), dim3(threads), 0, s, a, b);
  else hipLaunchKernelGGL((reduce_norm_two_kernel<bf16_t, 4>), dim3(a.rows), dim3(threads), 0, s, a, b);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Normed copies of the embeddings (bf16, see launch_embed_norm): 256 threads per row, eight columns per load and thread, the row in
// registers (C pieces).  Memory traffic alone: 2 bytes read and 2 per copy written (the reduce kernel, a thread's columns four at a time
// and 1024 threads per row: 32768 x 8192, two copies 461 -> 289 us; with the rows left as fp32 beside them 598).
// ------------------------------------------------------------------------------------------------
template <int C>
__global__ __launch_bounds__(256) void embed_norm_kernel(const bf16_t* __restrict__ emb, bf16_t* __restrict__ out_a, const bf16_t* __restrict__ gain_a,
                                                         bf16_t* __restrict__ out_b, const bf16_t* __restrict__ gain_b, int H, float eps) {
  const size_t base = (size_t)blockIdx.x * H;
  uint4 x[C];
  float ss = 0.f;
  auto unpack = [](const uint4 u, float (&f)[8]) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) { f[2 * e] = __uint_as_float(w[e] << 16); f[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u); }
  };
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = ((int)threadIdx.x + c * 256) * 8;
    x[c] = i < H ? load_16_at_8(emb + base + i) : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    float f[8];
    unpack(x[c], f);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += f[e] * f[e];
  }
  __shared__ float red[4];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float rs = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)H + eps);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = ((int)threadIdx.x + c * 256) * 8;
    if (i >= H) break;
    float f[8];
    unpack(x[c], f);
    auto store = [&](bf16_t* out, const bf16_t* gain) {
      float g[8];
      unpack(*reinterpret_cast<const uint4*>(gain + i), g);
      uint4 u;
      u.x = f32_to_bf16x2(f[0] * rs * g[0], f[1] * rs * g[1]);
      u.y = f32_to_bf16x2(f[2] * rs * g[2], f[3] * rs * g[3]);
      u.z = f32_to_bf16x2(f[4] * rs * g[4], f[5] * rs * g[5]);
      u.w = f32_to_bf16x2(f[6] * rs * g[6], f[7] * rs * g[7]);
      *reinterpret_cast<uint4*>(out + base + i) = u;
    };
    store(out_a, gain_a);
    if (out_b) store(out_b, gain_b);
  }
}

hipError_t launch_embed_norm(const bf16_t* emb, bf16_t* out_a, const bf16_t* gain_a, bf16_t* out_b, const bf16_t* gain_b, int rows, int H,
                             float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (H > EMBED_NORM_MAX_H || (H & 7) || !emb || !out_a || !gain_a || (out_b && !gain_b)) return hipErrorInvalidValue;
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(rows), dim3(256), 0, s, emb, out_a, gain_a, out_b, gain_b, H, eps); };
  if (H <= 4096) launch(embed_norm_kernel<2>);
  else if (H <= 8192) launch(embed_norm_kernel<4>);
  else launch(embed_norm_kernel<8>);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// The start of a pipeline stage (see StageInArgs), one workgroup per row, its C x 4 columns per thread in registers: memory traffic
// alone, 20 bytes per element where two passes of the reduce kernel moved 28 (4001 x 8192, bf16: 95 + 78 -> 112 us, 5.8 TB/s).
// ------------------------------------------------------------------------------------------------
template <typename T, int C>
__global__ __launch_bounds__(1024) void stage_in_kernel(StageInArgs a) {
  const int row = blockIdx.x, H = a.H, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const size_t base = (size_t)row * H;
  float p[C][4], v[C][4], sp = 0.f, sv = 0.f;   // x_{-1}, x_0 and their sums of squares
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = ((int)threadIdx.x + c * (int)blockDim.x) * 4;
    if (i >= H) break;
    float t[4], u[4];
    load4<float>(a.res + base + i, p[c]);
    if (a.att) load4<float>(a.att + base + i, t);
    if (a.mlp) load4<float>(a.mlp + base + i, u);
    for (int e = 0; e < 4; ++e) {
      if (a.att) p[c][e] += t[e];
      v[c][e] = a.mlp ? p[c][e] + u[e] : p[c][e];
    }
    store4<float>(a.x + base + i, v[c]);
    if (a.x_out) store4<float>(a.x_out + base + i, v[c]);
    sp += p[c][0] * p[c][0] + p[c][1] * p[c][1] + p[c][2] * p[c][2] + p[c][3] * p[c][3];
    sv += v[c][0] * v[c][0] + v[c][1] * v[c][1] + v[c][2] * v[c][2] + v[c][3] * v[c][3];
  }
  __shared__ float red[2][16];
  sp = wave_sum(sp);
  sv = wave_sum(sv);
  if ((threadIdx.x & 63) == 0) { red[0][wave] = sp; red[1][wave] = sv; }
  __syncthreads();
  sp = sv = 0.f;
  for (int w = 0; w < nw; ++w) { sp += red[0][w]; sv += red[1][w]; }
  const float rp = 1.0f / sqrtf(sp / (float)H + a.eps), rv = 1.0f / sqrtf(sv / (float)H + a.eps);
  auto normed = [&](void* out, const void* gain, int i, const float (&x)[4], float rs) {
    float g[4], y[4];
    load4<T>(reinterpret_cast<const T*>(gain) + i, g);
    for (int e = 0; e < 4; ++e) y[e] = x[e] * rs * g[e];
    store4<T>(reinterpret_cast<T*>(out) + base + i, y);
  };
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = ((int)threadIdx.x + c * (int)blockDim.x) * 4;
    if (i >= H) break;
    normed(a.out_a, a.gain_a, i, p[c], rp);
    normed(a.out_b, a.gain_b, i, v[c], rv);
  }
}

hipError_t launch_stage_in(const StageInArgs& a, bool is_bf16, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  if (a.H > STAGE_IN_MAX_H || !a.res || !a.x || !a.out_a || !a.gain_a || !a.out_b || !a.gain_b) return hipErrorInvalidValue;
  const int threads = a.H >= 4096 ? 1024 : 256;
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(a.rows), dim3(threads), 0, s, a); };
  if (a.H <= threads * 8) {   // (the registers of four are one workgroup per CU less)
    if (is_bf16) launch(stage_in_kernel<bf16_t, 2>);
    else launch(stage_in_kernel<float, 2>);
  } else if (is_bf16) {
    launch(stage_in_kernel<bf16_t, 4>);
  } else {
    launch(stage_in_kernel<float, 4>);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Plain projections: any size, both storage types, weights [K][N] as they were given, fp32 arithmetic.  One launch is
// one step of a module for ALL computed shards (grid z) and all the matrices that read the same rows (q | k | v, or gate
// and up), with what follows as its epilogue: a decode step of a small model is a chain of launches, and what counts is how
// many there are and how many memory round trips each one is long.  A workgroup takes MR rows x 64 columns and
// the whole K: 16 lanes side by side cover the columns, four at a time, and 16 groups of lanes deal out K in fours; every
// thread has 16 rows of the weights in flight before the activations are needed.  The groups' sums meet by lane
// exchange, the wavefronts' in LDS, in a fixed order.
// tiny fp32 model (hidden 256, 2 shards), one row: 22 us per matrix and shard (64 x 64 tiles, one k step of 16 in flight)
// -> 5 us for all
// of them; fp32 model of hidden 2048 (50 M weights a layer), 8 steps behind a prompt of 32: 23.9 -> 2.2 ms for 2 layers.
// Many rows, a layer of hidden 4096 and SwiGLU 11008, 64 x 64 tiles -> this, ms: fp32 128 / 512 / 2048 rows 4.6 / 7.4 / 40 ->
// 1.3 / 5.1 / 24.6, bf16 4.5 / 6.9 / 37 -> 1.3 / 4.8 / 19.8 (8.5 at 512 rows with the weights converted as they are loaded).
// ------------------------------------------------------------------------------------------------
// Blocks beyond what one grid dimension takes (fewer than 2^32 threads) go on in the second one, in rows of 2^20; the kernel leaves
// at once where its index is past the end.  (The row's length is a constant: gridDim comes from an implicit argument in memory,
// 557 -> 606 us on the tiny fp32 model's prompt of 32 and 8 steps.)
constexpr int FLAT_SHIFT = 20;
__device__ __forceinline__ unsigned flat_block() { return (blockIdx.y << FLAT_SHIFT) + blockIdx.x; }
static dim3 flat_grid(long long blocks, int n_shards) {
  const long long row = 1ll << FLAT_SHIFT;
  return dim3((unsigned)(blocks < row ? blocks : row), (unsigned)((blocks + row - 1) / row), (unsigned)n_shards);
}

// four weights as they were loaded: converted where they are multiplied, because a conversion in front of the activations' loads
// would wait for the weights first, one memory round trip after the other
template <typename T, bool VEC> struct PlainW4;
template <bool VEC> struct PlainW4<float, VEC> {
  float v[4];
  __device__ __forceinline__ void value(float (&f)[4]) const { for (int e = 0; e < 4; ++e) f[e] = v[e]; }
};
template <> struct PlainW4<bf16_t, true> {
  uint2 v;
  __device__ __forceinline__ void value(float (&f)[4]) const {
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
  }
};
template <> struct PlainW4<bf16_t, false> {
  uint32_t v[4];
  __device__ __forceinline__ void value(float (&f)[4]) const { for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(v[e] << 16); }
};

template <typename T, bool VEC>
__device__ __forceinline__ PlainW4<T, VEC> plain_w4(const T* w, int k, int K, int n, int N) {
  PlainW4<T, VEC> r{};
  if constexpr (VEC) {   // (N is a multiple of 4: a thread's columns are all inside or all outside)
    if (k < K && n < N) r = *reinterpret_cast<const PlainW4<T, VEC>*>(__builtin_assume_aligned(w + (size_t)k * N + n, 4 * sizeof(T)));
  } else {
    for (int e = 0; e < 4; ++e)
      if (k < K && n + e < N) r.v[e] = w[(size_t)k * N + n + e];
  }
  return r;
}

// element (row, k) of MR rows of a StreamSum; every load of a group of four pieces is requested before the first is needed
template <typename T, int MR>
__device__ __forceinline__ void stream_rows(const StreamSum& a, int H, int m0, int M, int k, float (&v)[MR]) {
  size_t at[MR];
#pragma unroll
  for (int m = 0; m < MR; ++m) {
    at[m] = (size_t)min(m0 + m, M - 1) * H + k;
    v[m] = a.emb ? load_f<T>(reinterpret_cast<const T*>(a.emb) + at[m]) : a.base[at[m]];
  }
  auto add = [&](int n, auto piece) {
    for (int s0 = 0; s0 < n; s0 += 4) {
      float t[4][MR];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int m = 0; m < MR; ++m) t[j][m] = s0 + j < n ? piece(s0 + j, at[m]) : 0.f;   // (uniform)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int m = 0; m < MR; ++m) v[m] = s0 + j < n ? v[m] + t[j][m] : v[m];
    }
  };
  for (int i = 0; i < a.n_adds; ++i) {
    const float* const parts = a.parts[i];
    const T* const peers = reinterpret_cast<const T*>(a.peers[i]);
    add(a.n_parts, [&](int s, size_t o) { return parts[s * a.part_stride + o]; });
    add(peers ? a.n_peers : 0, [&](int s, size_t o) { return load_f<T>(peers + s * a.peer_stride + o); });
  }
}

// rows m0 .. m0 + MR - 1 of x times columns n .. n + 3 (per lane) of the NM matrices w; the sums over all K end up in `sum` [NM][MR][64].
// NORM: the rows are those of a.in times the gain; the factor 1/rms commutes with the product and is applied to the sums; store: this
// workgroup leaves the rows in a.x_store.
// made: nothing, or what leaves a single row of at most KC elements in xs[0] (beside the weights that have been requested) instead of x.
struct PlainRowsGiven {};
template <typename T, int MR, bool VEC, int KC, int NM, bool NORM, typename F>
__device__ __forceinline__ void plain_product(const PlainGemmArgs& a, const T* x, int m0, const T* const (&w)[NM], int N, int n0, bool store, float (*xs)[KC],
                                              float (*red)[MR][64], float (*sum)[MR][64], float (*red_ss)[4], const F& made) {
  constexpr bool MADE = !__is_same(F, PlainRowsGiven);
  static_assert(!MADE || (MR == 1 && !NORM), "one row, as it is");
  const int M = a.M, K = a.K;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int c4 = (lane & 15) * 4, kg = t >> 4;
  constexpr int PASSES = KC / 64, ROWS = 256 / KC;   // (rows of x that the workgroup's threads take side by side)
  static_assert(!NORM || ROWS == 1, "a thread per k");
  float acc[NM][MR][4] = {}, ss[MR] = {};
  for (int k0 = 0; k0 < K; k0 += KC) {
    PlainW4<T, VEC> wr[NM][PASSES][4];   // [matrix][pass][k]
#pragma unroll
    for (int j = 0; j < NM; ++j)
#pragma unroll
      for (int i = 0; i < PASSES; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) wr[j][i][e] = plain_w4<T, VEC>(w[j], k0 + i * 64 + kg * 4 + e, K, n0 + c4, N);
    if constexpr (NORM) {
      const int k = k0 + t, kc = min(k, K - 1);
      float v[MR];
      const float gain = load_f<T>(reinterpret_cast<const T*>(a.gain) + kc);
      stream_rows<T, MR>(a.in, K, m0, M, kc, v);
      if (k0 > 0) __syncthreads();   // the previous pass has been read
#pragma unroll
      for (int m = 0; m < MR; ++m) {
        const bool ok = m0 + m < M && k < K;
        if (ok && store) a.x_store[(size_t)(m0 + m) * K + k] = v[m];
        xs[m][t] = ok ? v[m] * gain : 0.f;
        ss[m] += ok ? v[m] * v[m] : 0.f;
      }
    } else if constexpr (MADE) {
      made(xs[0]);
    } else {
      if (k0 > 0) __syncthreads();   // the previous pass has been read
#pragma unroll
      for (int i = 0; i < MR; i += ROWS) {
        const int m = ROWS == 1 ? i : i + t / KC, k = ROWS == 1 ? t : t % KC;
        xs[m][k] = m0 + m < M && k0 + k < K ? load_f<T>(x + (size_t)(m0 + m) * K + k0 + k) : 0.f;
      }
    }
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < PASSES; ++i)
#pragma unroll
      for (int j = 0; j < NM; ++j) {
        float wv[4][4];   // [k][column]
#pragma unroll
        for (int e = 0; e < 4; ++e) wr[j][i][e].value(wv[e]);
#pragma unroll
        for (int m = 0; m < MR; ++m) {
          const float4 xv = *reinterpret_cast<const float4*>(&xs[m][i * 64 + kg * 4]);
#pragma unroll
          for (int c = 0; c < 4; ++c)
            acc[j][m][c] = fmaf(xv.w, wv[3][c], fmaf(xv.z, wv[2][c], fmaf(xv.y, wv[1][c], fmaf(xv.x, wv[0][c], acc[j][m][c]))));
        }
      }
  }
#pragma unroll
  for (int j = 0; j < NM; ++j)
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float v = acc[j][m][c];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (lane < 16) red[j * 4 + wave][m][c4 + c] = v;
      }
  if constexpr (NORM) {
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      const float v = wave_sum(ss[m]);
      if (lane == 0) red_ss[m][wave] = v;
    }
  }
  __syncthreads();
  for (int i = t; i < NM * MR * 64; i += 256) {
    const int j = i / (MR * 64), m = i / 64 % MR, c = i & 63;
    float v = red[j * 4][m][c] + red[j * 4 + 1][m][c] + red[j * 4 + 2][m][c] + red[j * 4 + 3][m][c];
    if constexpr (NORM) v *= 1.0f / sqrtf((red_ss[m][0] + red_ss[m][1] + red_ss[m][2] + red_ss[m][3]) / (float)K + a.eps);
    sum[j][m][c] = v;
  }
  __syncthreads();
}

// Which tile a block takes.  Where the blocks are more than the chip holds at once, PLAIN_GROUP row blocks share a column block
// back to back and each of the 8 XCDs, to which blocks go round robin, works through one stretch of that order, so that a column
// block's weights come from memory once per group and not once per row block, which the caches cannot hide where a matrix is larger
// than they are (hidden 8192, SwiGLU 28672, one layer, 512 / 1024 / 2048 rows, ms: 64 x 64 tiles before fp32 23.8 / 43.2 / 98.0, bf16
// 21.2 / 39.0 / 89.0; columns first 31.3 / 64.1 / 135.1, 44.5 / 89.7 / 181.2; this 21.0 / 42.5 / 92.5, 20.2 / 39.2 / 80.1).  Else columns
// first (all blocks run side by side; hidden 1024, 32 rows: 176 against 181 us).
constexpr unsigned PLAIN_GROUP = 64;
__device__ __forceinline__ bool plain_tile(unsigned id, unsigned row_blocks, unsigned col_blocks, unsigned& m_blk, unsigned& col_blk) {
  const unsigned total = row_blocks * col_blocks, total8 = total & ~7u;
  if (id >= total) return false;
  if (total <= 512) {
    m_blk = id / col_blocks;
    col_blk = id % col_blocks;
    return true;
  }
  const unsigned at = id < total8 ? (id & 7) * (total8 >> 3) + (id >> 3) : id;
  const unsigned group = at / (PLAIN_GROUP * col_blocks), in_group = at % (PLAIN_GROUP * col_blocks);
  const unsigned gm = min(PLAIN_GROUP, row_blocks - group * PLAIN_GROUP);
  m_blk = group * PLAIN_GROUP + in_group % gm;
  col_blk = in_group / gm;
  return true;
}

// NM = 2: gate and up in one sweep over K, and more loads in flight in the other projections too.  (Two workgroups per CU: without the bound the rows that fp32 sums and norms itself cost two registers too many
// for that; three layers of 264 - 512 workgroups of four rows, hidden 512 and 1024, 2 - 7 % slower than it was as separate kernels, with it 14 - 20 % faster.)
template <typename T, int MR, bool VEC, int KC, bool NORM, int NM, typename F = PlainRowsGiven>
__device__ __forceinline__ void plain_gemm_block(const PlainGemmArgs& a, unsigned id, const F& made = F()) {
  __shared__ __attribute__((aligned(16))) float xs[MR][KC];
  __shared__ float red[4 * NM][MR][64];
  __shared__ float sum[2][MR][64];
  __shared__ float red_ss[MR][4];
  const int t = threadIdx.x, shard = blockIdx.z;
  unsigned m_blk, col_blk;
  if (MR == 1) {   // (a single row: m_blk is 0 inside the grid; written this way the tiny fp32 model's steps take 558 us, as one comparison 568)
    m_blk = id / (unsigned)a.n_blocks;
    col_blk = id % (unsigned)a.n_blocks;
    if (m_blk >= (unsigned)a.M) return;
  } else if (!plain_tile(id, ((unsigned)a.M + MR - 1) / MR, (unsigned)a.n_blocks, m_blk, col_blk)) {
    return;
  }
  const int m0 = (int)m_blk * MR;
  int blk = (int)col_blk, mat = 0;   // the matrices' column blocks side by side (SwiGLU: the gate's; the up matrix goes along)
  while (a.epilogue != PLAIN_SWIGLU && mat + 1 < a.n_mat && blk >= (a.N[mat] + 63) / 64) { blk -= (a.N[mat] + 63) / 64; ++mat; }
  const int n0 = blk * 64, N = a.N[mat];
  const T* x = reinterpret_cast<const T*>(a.x) + shard * a.x_stride;
  auto weights = [&](int i) { return reinterpret_cast<const T*>(reinterpret_cast<const char*>(a.w[i]) + shard * a.w_stride); };
  const bool store = NORM && a.x_store && col_blk == 0 && shard == 0;
  if (NM == 2 && a.epilogue == PLAIN_SWIGLU) {
    const T* const w[2] = {weights(0), weights(1)};
    plain_product<T, MR, VEC, KC, 2, NORM>(a, x, m0, w, N, n0, store, xs, red, sum, red_ss, made);
  } else {
    const T* const w[1] = {weights(mat)};
    plain_product<T, MR, VEC, KC, 1, NORM>(a, x, m0, w, N, n0, store, xs, red, sum, red_ss, made);
    if (a.epilogue == PLAIN_SWIGLU) {
      const T* const up[1] = {weights(1)};
      plain_product<T, MR, VEC, KC, 1, NORM>(a, x, m0, up, N, n0, false, xs, red, sum + 1, red_ss, made);
    }
  }
  if (a.epilogue == PLAIN_OUT) {
    for (int i = t; i < MR * 64; i += 256) {
      const int m = m0 + (i >> 6), n = n0 + (i & 63);
      if (m < a.M && n < N) a.out[shard * a.out_stride + (size_t)m * N + n] = sum[0][i >> 6][i & 63];
    }
  } else if (a.epilogue == PLAIN_SWIGLU) {
    T* act = reinterpret_cast<T*>(a.act) + shard * a.act_stride;
    for (int i = t; i < MR * 64; i += 256) {
      const int m = m0 + (i >> 6), n = n0 + (i & 63);
      const float g = sum[0][i >> 6][i & 63], u = sum[1][i >> 6][i & 63];
      if (m < a.M && n < N) store_f<T>(act + (size_t)m * N + n, g / (1.0f + expf(-g)) * u);
    }
  } else {   // matrices q, k, v: rotary embedding of q and k (adjacent pairs), k and v to the cache (v transposed)
    const int half = a.d >> 1;
    for (int i = t; i < MR * 32; i += 256) {
      const int m = m0 + (i >> 5), n = n0 + 2 * (i & 31);
      if (m >= a.M || n >= N) continue;   // (N is a multiple of the even d)
      float e = sum[0][i >> 5][2 * (i & 31)], o = sum[0][i >> 5][2 * (i & 31) + 1];
      const int b = m / a.T, pos = a.pos0 + m % a.T, head = n / a.d, dim = n % a.d;
      if (mat < 2) {
        const float c = a.cos_tab[(size_t)pos * half + (dim >> 1)], sn = a.sin_tab[(size_t)pos * half + (dim >> 1)];
        const float re = e * c - o * sn;
        o = e * sn + o * c;
        e = re;
      }
      if (mat == 0) {
        T* q = reinterpret_cast<T*>(a.q_out) + shard * a.q_stride + (size_t)m * N + n;
        store_f<T>(q, e);
        store_f<T>(q + 1, o);
      } else if (mat == 1) {
        T* k = reinterpret_cast<T*>(reinterpret_cast<char*>(a.cache_k) + shard * a.cache_stride) + (((size_t)b * a.nkv + head) * a.max_seq + pos) * a.d + dim;
        store_f<T>(k, e);
        store_f<T>(k + 1, o);
      } else {
        T* v = reinterpret_cast<T*>(reinterpret_cast<char*>(a.cache_v) + shard * a.cache_stride) + (((size_t)b * a.nkv + head) * a.d + dim) * a.max_seq + pos;
        store_f<T>(v, e);
        store_f<T>(v + a.max_seq, o);
      }
    }
  }
}

template <typename T, int MR, bool VEC, int KC, bool NORM, int NM>
__global__ __launch_bounds__(256, 2) void plain_gemm_kernel(PlainGemmArgs a) {
  plain_gemm_block<T, MR, VEC, KC, NORM, NM>(a, flat_block());
}

// The first projections of a layer's two modules in one launch, where neither reads what the other one writes: a's blocks, then b's.  Each launch of a
// small model is as long as one workgroup's round trips (4 - 6 us), so what counts is how many follow one another.
template <typename T, int MR, bool VEC>
__global__ __launch_bounds__(256, 2) void plain_inputs_kernel(PlainGemmArgs a, PlainGemmArgs b) {
  const unsigned id = blockIdx.x, n_a = (unsigned)a.n_blocks * (((unsigned)a.M + MR - 1) / MR);
  if (id < n_a) plain_gemm_block<T, MR, VEC, 256, true, 2>(a, id);
  else plain_gemm_block<T, MR, VEC, 256, true, 2>(b, id - n_a);
}

static int plain_col_blocks(const PlainGemmArgs& a) {
  int n = 0;
  for (int i = 0; i < (a.epilogue == PLAIN_SWIGLU ? 1 : a.n_mat); ++i) n += (a.N[i] + 63) / 64;
  return n;
}
// four weights per load where every row of every matrix starts on such a boundary
static bool plain_vec(const PlainGemmArgs& a) {
  bool vec = (a.w_stride & 15) == 0;
  for (int i = 0; i < a.n_mat; ++i) vec = vec && plain_four_at_once(a.w[i], a.N[i]);
  return vec;
}

template <typename T, int MR>
static hipError_t launch_plain_gemm_t(PlainGemmArgs a, bool vec, hipStream_t s) {
  a.n_blocks = plain_col_blocks(a);
  const long long blocks = (long long)a.n_blocks * (((long long)a.M + MR - 1) / MR);
  if (blocks > 0x7fffffff || a.n_shards > 65535) return hipErrorInvalidValue;
  const dim3 grid = flat_grid(blocks, a.n_shards);
  // k per pass: 256, or 128 where fp32 tiles of 16 rows are more than two workgroups per CU: their registers then allow three
  // (hidden 8192, 1024 rows 50.4 -> 42.5 ms; but hidden 1024, 128 rows, which do not fill two, 477 -> 583 us).  Same order of sums.
  auto launch = [&](auto kernel_vec, auto kernel) {
    if (vec) hipLaunchKernelGGL(kernel_vec, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a);
    return hipGetLastError();
  };
  if constexpr (MR == 16) {
    if constexpr (sizeof(T) == 4)
      if (blocks * a.n_shards > PLAIN_HELD_WORKGROUPS) return launch(plain_gemm_kernel<T, MR, true, 128, false, 1>, plain_gemm_kernel<T, MR, false, 128, false, 1>);
    return launch(plain_gemm_kernel<T, MR, true, 256, false, 1>, plain_gemm_kernel<T, MR, false, 256, false, 1>);
  } else {
    if (a.gain) return launch(plain_gemm_kernel<T, MR, true, 256, true, 2>, plain_gemm_kernel<T, MR, false, 256, true, 2>);
    // Gate and up in one sweep take the registers of two workgroups per CU, one after the other those of four, which is what counts where
    // there are more, beside the other module's on a second stream too (hidden 1024, 2 layers of 2 shards, 64 rows, one sweep / two: inter 1408
    // fp32 191 / 165 us, bf16 189 / 171; inter 2816 259 / 240, 249 / 217), and bf16 weights that come one by one are requested faster than they
    // can be waited for (inter 1409, 8 rows 329 / 310).
    if (blocks * a.n_shards <= a.held && (vec || sizeof(T) == 4)) return launch(plain_gemm_kernel<T, MR, true, 256, false, 2>, plain_gemm_kernel<T, MR, false, 256, false, 2>);
    return launch(plain_gemm_kernel<T, MR, true, 256, false, 1>, plain_gemm_kernel<T, MR, false, 256, false, 1>);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void stream_sum_kernel(StreamSum a, float* x_out, int rows, int H) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)rows * H) return;
  float v[1];
  stream_rows<T, 1>(a, H, (int)(i / H), rows, (int)(i % H), v);
  x_out[i] = v[0];
}

hipError_t launch_stream_sum(const StreamSum& a, float* x_out, int rows, int H, bool is_bf16, hipStream_t s) {
  const long long blocks = ((long long)rows * H + 255) / 256;
  if (blocks <= 0) return hipSuccess;
  if ((!a.emb && !a.base) || !x_out || blocks > 0x7fffff || a.n_adds < 0 || a.n_adds > 2) return hipErrorInvalidValue;
  if (is_bf16) hipLaunchKernelGGL(stream_sum_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, s, a, x_out, rows, H);
  else hipLaunchKernelGGL(stream_sum_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, s, a, x_out, rows, H);
  return hipGetLastError();
}

hipError_t launch_plain_gemm(const PlainGemmArgs& a, bool is_bf16, hipStream_t s) {
  if (a.M <= 0 || a.n_shards <= 0) return hipSuccess;
  if (a.gain && (a.M > PLAIN_NORM_ROWS || a.epilogue == PLAIN_OUT || (!a.in.emb && !a.in.base) || a.in.n_adds < 0 || a.in.n_adds > 2)) return hipErrorInvalidValue;
  const bool vec = plain_vec(a);
  // rows per workgroup: one for a single row; four for a few; more re-use of the weights beyond
  const int mr = a.M == 1 ? 1 : a.M <= PLAIN_NORM_ROWS ? 4 : 16;
  if (is_bf16) return mr == 1 ? launch_plain_gemm_t<bf16_t, 1>(a, vec, s) : mr == 4 ? launch_plain_gemm_t<bf16_t, 4>(a, vec, s) : launch_plain_gemm_t<bf16_t, 16>(a, vec, s);
  return mr == 1 ? launch_plain_gemm_t<float, 1>(a, vec, s) : mr == 4 ? launch_plain_gemm_t<float, 4>(a, vec, s) : launch_plain_gemm_t<float, 16>(a, vec, s);
}

// ------------------------------------------------------------------------------------------------
// Rotary embedding of q and k (adjacent pairs, angle = position * theta^(-2j/d), cos/sin from a
// host-made table) and append of k, v to the cache (packed-weight path, bf16).  One thread per pair.
// ------------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void rope_append_block(const RopeAppendArgs& a, unsigned block) {
  const int half = a.d >> 1;
  const int per_row = (a.nq + 2 * a.nkv) * half;
  const int rows = a.B * a.T;
  const long long gid = (long long)block * 256 + threadIdx.x;
  if (gid >= (long long)rows * per_row) return;
  const int row = (int)(gid / per_row);
  const int u = (int)(gid % per_row);
  const int b = row / a.T, t = row % a.T;
  const int pos0 = a.pos_dev ? *a.pos_dev : a.pos0;
  const int pos = pos0 + t;
  const int nqkv = (a.nq + 2 * a.nkv) * a.d;
  const int head = u / half, j = u % half;  // head index over q heads, then k heads, then v heads
  const int col = head * a.d + 2 * j;
  const float c = a.cos_tab[(size_t)pos * half + j], sn = a.sin_tab[(size_t)pos * half + j];   // (v does not need them)
  float e = 0.f, o = 0.f;
  four_at_a_time(a.n_parts, [&](int s, auto pieces) {
    constexpr int N = decltype(pieces)::n;
    float t[N][2];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const float* p = a.qkv + (s + k) * a.part_stride + (size_t)row * nqkv + col;
      t[k][0] = p[0];
      t[k][1] = p[1];
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
      e += t[k][0];
      o += t[k][1];
    }
  });
  if (head < a.nq + a.nkv) {
    const float re = fmaf(e, c, -(o * sn)), ro = fmaf(o, c, e * sn);   // (written out: every kernel around it gives the same bits)
    e = re;
    o = ro;
  }
  T* dst;
  if (head < a.nq) {
    dst = reinterpret_cast<T*>(a.q_out) + (size_t)row * a.nq * a.d + head * a.d + 2 * j;
  } else {
    const bool is_k = head < a.nq + a.nkv;
    if (!is_k) {  // V is kept transposed: [b][kv head][dim][position]
      const int kvh = head - a.nq - a.nkv;
      T* vt = reinterpret_cast<T*>(a.cache_v) + (((size_t)b * a.nkv + kvh) * a.d + 2 * j) * a.max_seq + pos;
      store_f<T>(vt, e);
      store_f<T>(vt + a.max_seq, o);
      if (!a.pos_dev && t == a.T - 1) {   // (a prefill)
        clear_block(vt + 1, pos + 1, a.max_seq);
        clear_block(vt + a.max_seq + 1, pos + 1, a.max_seq);
      }
      return;
    }
    const int kvh = head - a.nq;
    dst = reinterpret_cast<T*>(a.cache_k) + (((size_t)b * a.nkv + kvh) * a.max_seq + pos) * a.d + 2 * j;
  }
  store_f<T>(dst, e);
  store_f<T>(dst + 1, o);
}

__global__ __launch_bounds__(256) void rope_append_kernel(RopeAppendArgs a) { rope_append_block<bf16_t>(a, blockIdx.x); }

static unsigned rope_append_blocks(const RopeAppendArgs& a) { return (unsigned)(((long long)a.B * a.T * (a.nq + 2 * a.nkv) * (a.d / 2) + 255) / 256); }

hipError_t launch_rope_append(const RopeAppendArgs& a, hipStream_t s) {
  const unsigned blocks = rope_append_blocks(a);
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(rope_append_kernel, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Plain attention, any even head size up to 256: one workgroup per (row, q head, shard).  Its 4 wavefronts take chunks of
// 64 visible positions in turn, each with its own running softmax, and merge in LDS.  In a chunk a lane first owns a
// position (it walks that K row, 16 bytes at a time) and then a dim (it walks that row of the transposed V cache), so that
// every load is a whole piece of a row and a chunk is two memory round trips long, not one per position.
// tiny fp32 model, one row behind 32 positions: 23 us per shard -> 5.7 for both.
// ------------------------------------------------------------------------------------------------
template <typename T, bool VEC>
__device__ __forceinline__ void attn_generic_block(const AttnGenericArgs& a, unsigned unit) {
  __shared__ float qs[256];
  __shared__ __attribute__((aligned(16))) float ps[4][64];
  __shared__ float om[4][256], ms[4], ls[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (unit >= (unsigned)a.B * (unsigned)a.T * (unsigned)a.nq) return;
  const int row = (int)(unit / (unsigned)a.nq), h = (int)(unit % (unsigned)a.nq), shard = blockIdx.z;
  const int b = row / a.T, t = row % a.T;
  const int kvh = h / (a.nq / a.nkv);
  const int n_vis = a.pos0 + t + 1;
  const T* q = reinterpret_cast<const T*>(a.q) + shard * a.q_stride + (size_t)row * a.nq * a.d + h * a.d;
  const T* kb = reinterpret_cast<const T*>(reinterpret_cast<const char*>(a.cache_k) + shard * a.cache_stride) + ((size_t)b * a.nkv + kvh) * a.max_seq * a.d;
  const T* vb = reinterpret_cast<const T*>(reinterpret_cast<const char*>(a.cache_v) + shard * a.cache_stride) + ((size_t)b * a.nkv + kvh) * a.max_seq * a.d;
  if ((int)threadIdx.x < a.d) qs[threadIdx.x] = load_f<T>(q + threadIdx.x);
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)a.d);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float mx = -INFINITY, l = 0.f;
  for (int c0 = wave * 64; c0 < n_vis; c0 += 256) {
    const int n = min(64, n_vis - c0);
    float sc = -INFINITY;
    if (lane < n) {
      const T* kr = kb + (size_t)(c0 + lane) * a.d;
      float part[4] = {0.f, 0.f, 0.f, 0.f};
      if (VEC) {
#pragma unroll 8
        for (int i = 0; i < a.d; i += 4) {
          float kv[4];
          load4<T>(kr + i, kv);
          for (int e = 0; e < 4; ++e) part[e] = fmaf(qs[i + e], kv[e], part[e]);
        }
      } else {
        for (int i = 0; i < a.d; ++i) part[i & 3] = fmaf(qs[i], load_f<T>(kr + i), part[i & 3]);
      }
      sc = ((part[0] + part[1]) + (part[2] + part[3])) * scale;
    }
    const float mn = fmaxf(mx, wave_max(sc));
    const float ref = mn == -INFINITY ? 0.f : mn;   // (scores that are all -inf weigh nothing, they must not become NaN)
    const float corr = expf(mx - ref), p = lane < n ? expf(sc - ref) : 0.f;
    l = l * corr + wave_sum(p);
    mx = mn;
    ps[wave][lane] = p;
    __builtin_amdgcn_wave_barrier();   // (the wavefront's own LDS accesses stay in order)
    for (int e = 0; e < 4; ++e) {
      const int i = lane + 64 * e;
      if (i >= a.d) break;
      const T* vr = vb + (size_t)i * a.max_seq + c0;   // (the capacity and c0 are multiples of 64)
      float o[4] = {0.f, 0.f, 0.f, 0.f};
      int j = 0;
#pragma unroll 8
      for (; j + 4 <= n; j += 4) {
        float v[4];
        load4<T>(vr + j, v);
        for (int u = 0; u < 4; ++u) o[u] = fmaf(ps[wave][j + u], v[u], o[u]);
      }
      for (; j < n; ++j) o[0] = fmaf(ps[wave][j], load_f<T>(vr + j), o[0]);
      acc[e] = acc[e] * corr + ((o[0] + o[1]) + (o[2] + o[3]));
    }
    __builtin_amdgcn_wave_barrier();
  }
  for (int e = 0; e < 4; ++e)
    if (lane + 64 * e < a.d) om[wave][lane + 64 * e] = acc[e];
  if (lane == 0) { ms[wave] = mx; ls[wave] = l; }
  __syncthreads();
  if ((int)threadIdx.x < a.d) {
    const float m = fmaxf(fmaxf(ms[0], ms[1]), fmaxf(ms[2], ms[3]));   // (wavefront 0 always has a chunk)
    float o = 0.f, tot = 0.f;
    for (int w = 0; w < 4; ++w) {
      const float f = expf(ms[w] - m);
      o += om[w][threadIdx.x] * f;
      tot += ls[w] * f;
    }
    store_f<T>(reinterpret_cast<T*>(a.o) + shard * a.q_stride + (size_t)row * a.nq * a.d + h * a.d + threadIdx.x, o / tot);
  }
}

template <typename T, bool VEC>
__global__ __launch_bounds__(256) void attn_generic_kernel(AttnGenericArgs a) {
  attn_generic_block<T, VEC>(a, flat_block());
}

// The attention of a layer and the last projection of its MLP in one launch (the MLP's first one has run beside the QKV projection)
template <typename T, int MR, bool VEC_A, bool VEC_B>
__global__ __launch_bounds__(256, 2) void plain_attn_beside_kernel(AttnGenericArgs a, PlainGemmArgs b) {
  const unsigned id = blockIdx.x, n_a = (unsigned)a.B * (unsigned)a.T * (unsigned)a.nq;
  if (id < n_a) attn_generic_block<T, VEC_A>(a, id);
  else plain_gemm_block<T, MR, VEC_B, 256, false, 2>(b, id - n_a);
}

// One row's attention over all nq (1, 2 or 4) heads of a computed shard, as every workgroup of its output projection needs it: out[nq * d], rounded to T
// as the stored one is.  The wavefronts are dealt out over the heads and then over chunks of 64 positions; a chunk as in attn_generic_block.
template <typename T, bool VEC>
__device__ __forceinline__ void attn_one_row(const AttnGenericArgs& a, int shard, float* out) {
  __shared__ float qs[256];
  __shared__ __attribute__((aligned(16))) float ps[4][64];
  __shared__ float om[4][256], ms[4], ls[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nqd = a.nq * a.d;
  const int h = wave % a.nq, first = wave / a.nq, stride = 4 / a.nq;
  const int n_vis = a.pos0 + 1;
  const T* kb = reinterpret_cast<const T*>(reinterpret_cast<const char*>(a.cache_k) + shard * a.cache_stride) + (size_t)(h / (a.nq / a.nkv)) * a.max_seq * a.d;
  const T* vb = reinterpret_cast<const T*>(reinterpret_cast<const char*>(a.cache_v) + shard * a.cache_stride) + (size_t)(h / (a.nq / a.nkv)) * a.max_seq * a.d;
  if ((int)threadIdx.x < nqd) qs[threadIdx.x] = load_f<T>(reinterpret_cast<const T*>(a.q) + shard * a.q_stride + threadIdx.x);
  __syncthreads();
  const float* const qh = qs + h * a.d;
  const float scale = 1.0f / sqrtf((float)a.d);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float mx = -INFINITY, l = 0.f;
  for (int c0 = first * 64; c0 < n_vis; c0 += stride * 64) {
    const int n = min(64, n_vis - c0);
    float sc = -INFINITY;
    if (lane < n) {
      const T* kr = kb + (size_t)(c0 + lane) * a.d;
      float part[4] = {0.f, 0.f, 0.f, 0.f};
      if (VEC) {
#pragma unroll 8
        for (int i = 0; i < a.d; i += 4) {
          float kv[4];
          load4<T>(kr + i, kv);
          for (int e = 0; e < 4; ++e) part[e] = fmaf(qh[i + e], kv[e], part[e]);
        }
      } else {
        for (int i = 0; i < a.d; ++i) part[i & 3] = fmaf(qh[i], load_f<T>(kr + i), part[i & 3]);
      }
      sc = ((part[0] + part[1]) + (part[2] + part[3])) * scale;
    }
    const float mn = fmaxf(mx, wave_max(sc));
    const float ref = mn == -INFINITY ? 0.f : mn;   // (scores that are all -inf weigh nothing, they must not become NaN)
    const float corr = expf(mx - ref), p = lane < n ? expf(sc - ref) : 0.f;
    l = l * corr + wave_sum(p);
    mx = mn;
    ps[wave][lane] = p;
    __builtin_amdgcn_wave_barrier();   // (the wavefront's own LDS accesses stay in order)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = lane + 64 * e;
      if (i >= a.d) continue;
      const T* vr = vb + (size_t)i * a.max_seq + c0;   // (the capacity and c0 are multiples of 64)
      float o[4] = {0.f, 0.f, 0.f, 0.f};
      int j = 0;
#pragma unroll 8
      for (; j + 4 <= n; j += 4) {
        float v[4];
        load4<T>(vr + j, v);
        for (int u = 0; u < 4; ++u) o[u] = fmaf(ps[wave][j + u], v[u], o[u]);
      }
      for (; j < n; ++j) o[0] = fmaf(ps[wave][j], load_f<T>(vr + j), o[0]);
      acc[e] = acc[e] * corr + ((o[0] + o[1]) + (o[2] + o[3]));
    }
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (lane + 64 * e < a.d) om[wave][lane + 64 * e] = acc[e];
  if (lane == 0) { ms[wave] = mx; ls[wave] = l; }
  __syncthreads();
  const int t = threadIdx.x;
  float res = 0.f;
  if (t < nqd) {
    const int head = t / a.d, dim = t % a.d;
    float m = ms[head], o = 0.f, tot = 0.f;   // (the head's first wavefront always has a chunk)
    for (int w = head + a.nq; w < 4; w += a.nq) m = fmaxf(m, ms[w]);
    const float ref = m == -INFINITY ? 0.f : m;
    for (int w = head; w < 4; w += a.nq) {
      const float f = expf(ms[w] - ref);
      o += om[w][dim] * f;
      tot += ls[w] * f;
    }
    T r;
    store_f<T>(&r, o / tot);
    res = load_f<T>(&r);
  }
  out[t] = res;   // (a pass of 256 elements: zeros behind the row)
}

// One row: the attention and its output projection (every workgroup of o makes the attention's output itself, which is little where the cache is short) beside the
// last projection of the MLP
template <typename T, bool VEC_A, bool VEC>
__global__ __launch_bounds__(256, 2) void plain_attn_out_kernel(AttnGenericArgs a, PlainGemmArgs o, PlainGemmArgs b) {
  const unsigned id = blockIdx.x;
  if (id < (unsigned)o.n_blocks)
    plain_gemm_block<T, 1, VEC, 256, false, 1>(o, id, [&](float* xs) { attn_one_row<T, VEC_A>(a, blockIdx.z, xs); });
  else plain_gemm_block<T, 1, VEC, 256, false, 2>(b, id - (unsigned)o.n_blocks);
}
template <typename T>
static hipError_t launch_plain_attn_out_t(const AttnGenericArgs& a, const PlainGemmArgs& o, const PlainGemmArgs& b, bool vec_a, bool vec, dim3 grid, hipStream_t s) {
  if (vec_a && vec) hipLaunchKernelGGL((plain_attn_out_kernel<T, true, true>), grid, dim3(256), 0, s, a, o, b);
  else if (vec_a) hipLaunchKernelGGL((plain_attn_out_kernel<T, true, false>), grid, dim3(256), 0, s, a, o, b);
  else if (vec) hipLaunchKernelGGL((plain_attn_out_kernel<T, false, true>), grid, dim3(256), 0, s, a, o, b);
  else hipLaunchKernelGGL((plain_attn_out_kernel<T, false, false>), grid, dim3(256), 0, s, a, o, b);
  return hipGetLastError();
}

template <typename T, int MR>
static hipError_t launch_plain_inputs_t(const PlainGemmArgs& a, const PlainGemmArgs& b, bool vec, dim3 grid, hipStream_t s) {
  if (vec) hipLaunchKernelGGL((plain_inputs_kernel<T, MR, true>), grid, dim3(256), 0, s, a, b);
  else hipLaunchKernelGGL((plain_inputs_kernel<T, MR, false>), grid, dim3(256), 0, s, a, b);
  return hipGetLastError();
}
template <typename T, int MR>
static hipError_t launch_plain_attn_beside_t(const AttnGenericArgs& a, const PlainGemmArgs& b, bool vec_a, bool vec_b, dim3 grid, hipStream_t s) {
  if (vec_a && vec_b) hipLaunchKernelGGL((plain_attn_beside_kernel<T, MR, true, true>), grid, dim3(256), 0, s, a, b);
  else if (vec_a) hipLaunchKernelGGL((plain_attn_beside_kernel<T, MR, true, false>), grid, dim3(256), 0, s, a, b);
  else if (vec_b) hipLaunchKernelGGL((plain_attn_beside_kernel<T, MR, false, true>), grid, dim3(256), 0, s, a, b);
  else hipLaunchKernelGGL((plain_attn_beside_kernel<T, MR, false, false>), grid, dim3(256), 0, s, a, b);
  return hipGetLastError();
}

// Both launches together hold at most PLAIN_HELD_WORKGROUPS workgroups, two per CU; of a bf16 matrix whose weights come one by one (gain: the
// caller has asked) the kernels by themselves know a better way
bool plain_beside(const PlainGemmArgs& qkv, const AttnGenericArgs& attn, const PlainGemmArgs& gate_up, const PlainGemmArgs& down, bool is_bf16) {
  const int rows = qkv.M, shards = qkv.n_shards;
  if (rows < 1 || rows > PLAIN_NORM_ROWS || shards < 1 || !qkv.gain || !gate_up.gain || attn.d > 256) return false;
  if (is_bf16 && !(plain_vec(qkv) && plain_vec(gate_up) && plain_vec(down))) return false;
  const long long first = plain_workgroups(rows, plain_col_blocks(qkv) + plain_col_blocks(gate_up), shards);
  const long long second = (long long)rows * attn.nq * shards + plain_workgroups(rows, plain_col_blocks(down), shards);
  return first <= PLAIN_HELD_WORKGROUPS && second <= PLAIN_HELD_WORKGROUPS;
}
// A single row whose heads' outputs are one pass of the projection, behind a cache of one chunk per wavefront, so that the sums are those of the attention by
// itself (tiny fp32 model, prompt of 32 and 8 steps 306 -> 280 us; hidden 512 463 -> 407, bf16 458 -> 389; behind 300 positions, several chunks, 325 -> 361).
bool plain_attn_out_fits(const AttnGenericArgs& a, const PlainGemmArgs& o, const PlainGemmArgs& down, bool is_bf16) {
  if (a.B != 1 || a.T != 1 || (a.nq != 1 && a.nq != 2 && a.nq != 4) || a.nq * a.d > 256 || o.K != a.nq * a.d || o.M != 1 || down.M != 1) return false;
  if (is_bf16 && !(plain_vec(o) && plain_vec(down))) return false;
  return (long long)(a.pos0 + 1) * a.nq <= PLAIN_ATTN_OUT_POSITIONS && (long long)(plain_col_blocks(o) + plain_col_blocks(down)) * a.n_shards <= PLAIN_HELD_WORKGROUPS;
}
hipError_t launch_plain_attn_out(const AttnGenericArgs& a, PlainGemmArgs o, PlainGemmArgs b, bool is_bf16, hipStream_t s) {
  if (!plain_attn_out_fits(a, o, b, is_bf16) || a.n_shards <= 0 || a.n_shards != o.n_shards || a.n_shards != b.n_shards) return hipErrorInvalidValue;
  o.n_blocks = plain_col_blocks(o);
  b.n_blocks = plain_col_blocks(b);
  const bool vec_a = a.d % 4 == 0, vec = plain_vec(o) && plain_vec(b);
  const dim3 grid((unsigned)(o.n_blocks + b.n_blocks), 1, (unsigned)a.n_shards);
  return is_bf16 ? launch_plain_attn_out_t<bf16_t>(a, o, b, vec_a, vec, grid, s) : launch_plain_attn_out_t<float>(a, o, b, vec_a, vec, grid, s);
}
hipError_t launch_plain_inputs(PlainGemmArgs a, PlainGemmArgs b, bool is_bf16, hipStream_t s) {
  if (a.M <= 0 || a.M > PLAIN_NORM_ROWS || b.M != a.M || a.n_shards <= 0 || b.n_shards != a.n_shards || !a.gain || !b.gain) return hipErrorInvalidValue;
  a.n_blocks = plain_col_blocks(a);
  b.n_blocks = plain_col_blocks(b);
  const bool vec = plain_vec(a) && plain_vec(b), one = a.M == 1;
  const dim3 grid((unsigned)((a.n_blocks + b.n_blocks) * (one ? 1 : (a.M + 3) / 4)), 1, (unsigned)a.n_shards);
  if (is_bf16) return one ? launch_plain_inputs_t<bf16_t, 1>(a, b, vec, grid, s) : launch_plain_inputs_t<bf16_t, 4>(a, b, vec, grid, s);
  return one ? launch_plain_inputs_t<float, 1>(a, b, vec, grid, s) : launch_plain_inputs_t<float, 4>(a, b, vec, grid, s);
}
hipError_t launch_plain_attn_beside(const AttnGenericArgs& a, PlainGemmArgs b, bool is_bf16, hipStream_t s) {
  const int rows = a.B * a.T;
  if (rows <= 0 || rows > PLAIN_NORM_ROWS || b.M != rows || a.n_shards <= 0 || b.n_shards != a.n_shards || a.d > 256) return hipErrorInvalidValue;
  b.n_blocks = plain_col_blocks(b);
  const bool vec_a = a.d % 4 == 0, vec_b = plain_vec(b), one = rows == 1;
  const dim3 grid((unsigned)(rows * a.nq + b.n_blocks * (one ? 1 : (rows + 3) / 4)), 1, (unsigned)a.n_shards);
  if (is_bf16) return one ? launch_plain_attn_beside_t<bf16_t, 1>(a, b, vec_a, vec_b, grid, s) : launch_plain_attn_beside_t<bf16_t, 4>(a, b, vec_a, vec_b, grid, s);
  return one ? launch_plain_attn_beside_t<float, 1>(a, b, vec_a, vec_b, grid, s) : launch_plain_attn_beside_t<float, 4>(a, b, vec_a, vec_b, grid, s);
}

hipError_t launch_attn_generic(const AttnGenericArgs& a, bool is_bf16, hipStream_t s) {
  const long long units = (long long)a.B * a.T * a.nq;
  if (units <= 0 || a.n_shards <= 0) return hipSuccess;
  if (units > 0x7fffffff || a.n_shards > 65535 || a.d > 256) return hipErrorInvalidValue;
  const dim3 grid = flat_grid(units, a.n_shards);
  const bool vec = a.d % 4 == 0;   // (a K row then starts on a boundary of four elements)
  if (is_bf16) {
    if (vec) hipLaunchKernelGGL((attn_generic_kernel<bf16_t, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((attn_generic_kernel<bf16_t, false>), grid, dim3(256), 0, s, a);
  } else {
    if (vec) hipLaunchKernelGGL((attn_generic_kernel<float, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((attn_generic_kernel<float, false>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// SwiGLU of a split gate/up projection (packed-weight path).
// Four activations per thread; the gate columns of eight activations and the matching up columns are neighbours.
__device__ __forceinline__ void swiglu_parts_block(const SwigluPartsArgs& a, unsigned block) {
  const long long gid = (long long)block * 256 + threadIdx.x;
  const int i4 = a.I >> 2;
  if (gid >= (long long)a.M * i4) return;
  const int m = (int)(gid / i4), i = (int)(gid % i4) * 4;
  const float* p = a.parts + (size_t)m * 2 * a.I + 16 * (i >> 3) + (i & 7);
  float g[4] = {}, u[4] = {}, y[4];
  four_at_a_time(a.n_parts, [&](int s, auto pieces) {
    constexpr int N = decltype(pieces)::n;
    float t[N][2][4];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      load4<float>(p + (s + k) * a.part_stride, t[k][0]);
      load4<float>(p + (s + k) * a.part_stride + 8, t[k][1]);
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
      for (int e = 0; e < 4; ++e) { g[e] += t[k][0][e]; u[e] += t[k][1][e]; }
  });
  for (int e = 0; e < 4; ++e) y[e] = g[e] / (1.0f + __expf(-g[e])) * u[e];
  store4<bf16_t>(a.act + (size_t)m * a.I + i, y);
}

__global__ __launch_bounds__(256) void swiglu_parts_kernel(SwigluPartsArgs a) { swiglu_parts_block(a, blockIdx.x); }

// Rotary + append and SwiGLU of a layer whose modules share launches: neither reads what the other writes, and each by itself is as long as its round trips
__global__ __launch_bounds__(256) void rope_swiglu_kernel(RopeAppendArgs a, SwigluPartsArgs b, unsigned n_a) {
  if (blockIdx.x < n_a) rope_append_block<bf16_t>(a, blockIdx.x);
  else swiglu_parts_block(b, blockIdx.x - n_a);
}

static unsigned swiglu_parts_blocks(const SwigluPartsArgs& a) { return (unsigned)(((long long)a.M * (a.I >> 2) + 255) / 256); }

hipError_t launch_swiglu_parts(const SwigluPartsArgs& a, hipStream_t s) {
  const unsigned blocks = swiglu_parts_blocks(a);
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(swiglu_parts_kernel, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_rope_swiglu(const RopeAppendArgs& a, const SwigluPartsArgs& b, hipStream_t s) {
  const unsigned n_a = rope_append_blocks(a), n_b = swiglu_parts_blocks(b);
  if (!(n_a + n_b)) return hipSuccess;
  hipLaunchKernelGGL(rope_swiglu_kernel, dim3(n_a + n_b), dim3(256), 0, s, a, b, n_a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Caller-made cache content [B][nkv][S][d] -> K cache rows, V cache transposed.
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ void load_kv_kernel(const T* __restrict__ k, const T* __restrict__ v, T* __restrict__ ck,
                               T* __restrict__ cv, int B, int nkv, int S, int d, int max_seq, bool clear) {
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = (long long)B * nkv * S * d;
  if (gid >= total) return;
  const int i = (int)(gid % d);
  const int p = (int)((gid / d) % S);
  const long long bh = gid / ((long long)d * S);
  ck[((size_t)bh * max_seq + p) * d + i] = k[gid];
  T* const at = cv + ((size_t)bh * d + i) * max_seq + p;
  *at = v[gid];
  if (clear && p == S - 1) clear_block(at + 1, S, max_seq);
}

// The same, 16 bytes per lane on both sides: a workgroup takes P positions of one (sequence, kv head), copies its K rows
// and turns its V rows in LDS, so that a store covers whole pieces of a cache row.  (Element by element every V value is
// a memory transaction of its own.)
// Measured, us per layer: 64 sequences x 8 kv heads x 1024 positions 435 -> 102 (5.3 TB/s read + written);
// 16 x 8 x 1024 115 -> 29; 4 x 1 x 32001 117 -> 28.
template <typename T, int P>
__global__ __launch_bounds__(256) void load_kv_tiles_kernel(const T* __restrict__ k, const T* __restrict__ v, T* __restrict__ ck,
                                                            T* __restrict__ cv, int S, int d, int max_seq, bool clear) {
  constexpr int E = 16 / sizeof(T);            // elements per 16 bytes
  constexpr int ROW = P + 4 / (int)sizeof(T);  // a turned row: one word of padding
  extern __shared__ __attribute__((aligned(16))) unsigned char load_kv_lds[];
  T* const turned = reinterpret_cast<T*>(load_kv_lds);   // [d][ROW]
  const int p0 = blockIdx.x * P, n = min(P, S - p0);
  const size_t bh = blockIdx.y;
  const int segs = d / E;
  const T* ks = k + (bh * S + p0) * d;
  const T* vs = v + (bh * S + p0) * d;
  T* kd = ck + (bh * max_seq + p0) * d;
  for (int i = threadIdx.x; i < n * segs; i += 256) {
    *reinterpret_cast<uint4*>(kd + (size_t)i * E) = *reinterpret_cast<const uint4*>(ks + (size_t)i * E);
    const uint4 u = *reinterpret_cast<const uint4*>(vs + (size_t)i * E);
    const T* e = reinterpret_cast<const T*>(&u);
    const int p = i / segs, dim = i % segs * E;
#pragma unroll
    for (int j = 0; j < E; ++j) turned[(dim + j) * ROW + p] = e[j];
  }
  __syncthreads();
  const int pieces = P / E;
  // the last tile is stored as whole cache lines, zeros behind the last position (16 x 8 x 1023 positions: 31 -> 24 us); one that
  // ends with its lines clears the next ones where asked to
  if (n < P || (clear && p0 + P == S && S < max_seq)) {
    const int from = n < P ? (n + E - 1) / E * E : P, m = ((n < P ? P : 2 * P) - from) / E;   // (the rows are whole tiles long)
    for (int i = threadIdx.x; i < d * m; i += 256)
      *reinterpret_cast<uint4*>(cv + (bh * d + i / m) * max_seq + p0 + from + i % m * E) = make_uint4(0u, 0u, 0u, 0u);
  }
  for (int i = threadIdx.x; i < d * pieces; i += 256) {
    const int dim = i / pieces, p = i % pieces * E;
    if (p >= n) continue;
    T* dst = cv + (bh * d + dim) * max_seq + p0 + p;
    uint4 u;
    T* e = reinterpret_cast<T*>(&u);
#pragma unroll
    for (int j = 0; j < E; ++j) e[j] = turned[dim * ROW + p + j];
    if (p + E <= n) {
      *reinterpret_cast<uint4*>(dst) = u;   // (max_seq is a multiple of 128, p0 and p of E)
    } else {
      for (int j = 0; j < E; ++j) dst[j] = p + j < n ? e[j] : T(0);
    }
  }
}

template <typename T, int P>
static hipError_t launch_load_kv_tiles(const void* k, const void* v, void* ck, void* cv, int B, int nkv, int S, int d, int max_seq, bool clear, hipStream_t s) {
  const size_t lds = (size_t)d * (P + 4 / sizeof(T)) * sizeof(T);   // at most 36 KiB (d <= 256)
  hipLaunchKernelGGL((load_kv_tiles_kernel<T, P>), dim3((S + P - 1) / P, B * nkv), dim3(256), lds, s, (const T*)k, (const T*)v, (T*)ck, (T*)cv, S, d, max_seq, clear);
  return hipGetLastError();
}

hipError_t launch_load_kv(const void* k, const void* v, void* cache_k, void* cache_v, int B, int nkv, int S, int d,
                          int max_seq, bool is_bf16, bool clear, hipStream_t s) {
  const long long total = (long long)B * nkv * S * d;
  if (total <= 0) return hipSuccess;
  // 16-byte accesses: the caller's tensors have to be aligned and a row has to be whole pieces (d need only be even), and
  // the cache rows whole tiles (max_seq, a multiple of 128, and the library's own allocation); B * nkv is a grid dimension
  const bool aligned = (((uintptr_t)k | (uintptr_t)v) & 15) == 0 && d % (is_bf16 ? 8 : 4) == 0 && d <= 256 && max_seq % 64 == 0 && (long long)B * nkv <= 65535;
  if (aligned) return is_bf16 ? launch_load_kv_tiles<bf16_t, 64>(k, v, cache_k, cache_v, B, nkv, S, d, max_seq, clear, s)
                              : launch_load_kv_tiles<float, 32>(k, v, cache_k, cache_v, B, nkv, S, d, max_seq, clear, s);
  const unsigned blocks = (unsigned)((total + 255) / 256);
  if (is_bf16)
    hipLaunchKernelGGL(load_kv_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, (const bf16_t*)k, (const bf16_t*)v,
                       (bf16_t*)cache_k, (bf16_t*)cache_v, B, nkv, S, d, max_seq, clear);
  else
    hipLaunchKernelGGL(load_kv_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float*)k, (const float*)v,
                       (float*)cache_k, (float*)cache_v, B, nkv, S, d, max_seq, clear);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Generation head: token embedding (row gather), final RMSNorm, greedy sampling (first arg max).
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void embed_gather_kernel(const int* __restrict__ tokens, const T* __restrict__ table,
                                                           T* __restrict__ out, int H, int vocab, unsigned* bad_id) {
  const int r = blockIdx.x;
  const int raw = tokens[r];
  const int tok = min(max(raw, 0), vocab - 1);   // no access leaves the table; an id outside it is reported
  if (raw != tok && bad_id && threadIdx.x == 0) __hip_atomic_store(bad_id, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  for (int i = threadIdx.x; i < H; i += 256) out[(size_t)r * H + i] = table[(size_t)tok * H + i];
}

hipError_t launch_embed_gather(const int* tokens, const void* table, void* x_out, int rows, int H, int vocab,
                               unsigned* bad_id, bool is_bf16, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (is_bf16) hipLaunchKernelGGL(embed_gather_kernel<bf16_t>, dim3(rows), dim3(256), 0, s, tokens, (const bf16_t*)table, (bf16_t*)x_out, H, vocab, bad_id);
  else hipLaunchKernelGGL(embed_gather_kernel<float>, dim3(rows), dim3(256), 0, s, tokens, (const float*)table, (float*)x_out, H, vocab, bad_id);
  return hipGetLastError();
}

// (a thread's elements of a pass in registers: one round trip for 8192 columns of 1024 threads, which long rows take)
template <typename T, int THREADS>
__global__ __launch_bounds__(THREADS) void head_norm_kernel(const float* __restrict__ x, const T* __restrict__ gain,
                                                            T* __restrict__ y, int H, float eps, int tiled) {
  constexpr int N = 8;
  const auto at = [&](int i) { return tiled ? ((size_t)(i >> 3) * gridDim.x + blockIdx.x) * 8 + (i & 7) : (size_t)blockIdx.x * H + i; };
  __shared__ float part[THREADS / 64];
  const float* xr = x + (size_t)blockIdx.x * H;
  float v[N], ss = 0.f;
#pragma unroll
  for (int e = 0; e < N; ++e) v[e] = (int)threadIdx.x + e * THREADS < H ? xr[threadIdx.x + e * THREADS] : 0.f;
#pragma unroll
  for (int e = 0; e < N; ++e) ss = fmaf(v[e], v[e], ss);
  for (int i = threadIdx.x + N * THREADS; i < H; i += THREADS) ss = fmaf(xr[i], xr[i], ss);
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) ss += part[w];
  const float rs = 1.0f / sqrtf(ss / (float)H + eps);
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int i = threadIdx.x + e * THREADS;
    if (i < H) store_f(y + at(i), v[e] * rs * (gain ? load_f(gain + i) : 1.0f));
  }
  for (int i = threadIdx.x + N * THREADS; i < H; i += THREADS)
    store_f(y + at(i), xr[i] * rs * (gain ? load_f(gain + i) : 1.0f));
}

template <typename T>
static void launch_head_norm_t(const float* x, const void* gain, void* y, int rows, int H, float eps, bool tiled, hipStream_t s) {
  if (H > 2048) hipLaunchKernelGGL((head_norm_kernel<T, 1024>), dim3(rows), dim3(1024), 0, s, x, (const T*)gain, (T*)y, H, eps, tiled ? 1 : 0);
  else hipLaunchKernelGGL((head_norm_kernel<T, 256>), dim3(rows), dim3(256), 0, s, x, (const T*)gain, (T*)y, H, eps, tiled ? 1 : 0);
}
hipError_t launch_head_norm(const float* x, const void* gain, void* y, int rows, int H, float eps, bool tiled, bool is_bf16,
                            hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (tiled && (H & 7)) return hipErrorInvalidValue;
  if (is_bf16) launch_head_norm_t<bf16_t>(x, gain, y, rows, H, eps, tiled, s);
  else launch_head_norm_t<float>(x, gain, y, rows, H, eps, tiled, s);
  return hipGetLastError();
}

// A thread keeps the first maximum of its share (indices ascending), the merge prefers the lower index among equal values,
// so the result is the first arg max of the row; a NaN gives way to any number.
// What bounds it is how much of a row is in flight, so threads request 16 bytes four times over before they compare, and rows of
// ARGMAX_SPLIT_V logits and more are cut over ARGMAX_PARTS workgroups, whose picks a second kernel merges; they lie where the normed rows lay
// that the logits were made from.  16 rows of 128256 logits, one workgroup per row / cut: 12.5 / 4.9 + 4.6 us as the profiler has them, the whole
// head 205 / 193 with the norm's 1024 threads; 32000 logits, one row, 54.3 / 50.5; below that a row is one round trip either way.
// ------------------------------------------------------------------------------------------------
struct Pick {
  float best;
  int at;      // ARGMAX_NONE: none yet
};
constexpr int ARGMAX_NONE = 0x7fffffff;
__device__ __forceinline__ void pick_merge(Pick& p, float ov, int oi) {
  if (oi != ARGMAX_NONE && (p.at == ARGMAX_NONE || ov > p.best || (ov == p.best && oi < p.at) || (p.best != p.best && (ov == ov || oi < p.at)))) {
    p.best = ov;
    p.at = oi;
  }
}
// THREADS threads take the elements from .. to - 1 of a row (with vec both multiples of 4, except the row's end); the result is thread 0's
template <int THREADS>
__device__ __forceinline__ Pick pick_first_max(const float* __restrict__ lr, int from, int to, int vec) {
  __shared__ float bv[THREADS / 64];
  __shared__ int bi[THREADS / 64];
  Pick p{-INFINITY, ARGMAX_NONE};
  auto take = [&](float v, int i) {
    if (p.at == ARGMAX_NONE || v > p.best || p.best != p.best) { p.best = v; p.at = i; }   // strictly greater: the earliest index stays
  };
  if (vec) {
    const float4* l4 = reinterpret_cast<const float4*>(lr);
    const int n4 = to >> 2;
    for (int i0 = (from >> 2) + threadIdx.x; i0 < n4; i0 += 4 * THREADS) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = l4[min(i0 + u * THREADS, n4 - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * THREADS;
        if (i < n4) { take(v[u].x, 4 * i); take(v[u].y, 4 * i + 1); take(v[u].z, 4 * i + 2); take(v[u].w, 4 * i + 3); }
      }
    }
  } else {
    for (int i = from + threadIdx.x; i < to; i += THREADS) take(lr[i], i);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(p.best, o, 64);
    const int oi = __shfl_xor(p.at, o, 64);
    pick_merge(p, ov, oi);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { bv[wave] = p.best; bi[wave] = p.at; }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < THREADS / 64; ++w) pick_merge(p, bv[w], bi[w]);
  return p;
}

__global__ __launch_bounds__(1024) void argmax_kernel(const float* __restrict__ logits, int* __restrict__ out, int V, int vec) {
  const Pick p = pick_first_max<1024>(logits + (size_t)blockIdx.x * V, 0, V, vec);
  if (threadIdx.x == 0) out[blockIdx.x] = p.at == ARGMAX_NONE ? 0 : p.at;
}

#define ARGMAX_PARTS 16
#define ARGMAX_SPLIT_V 32000
__global__ __launch_bounds__(256) void argmax_part_kernel(const float* __restrict__ logits, Pick* __restrict__ picks, int V) {
  const int per = ((V + ARGMAX_PARTS - 1) / ARGMAX_PARTS + 3) & ~3, from = min(V, (int)blockIdx.x * per);
  const Pick p = pick_first_max<256>(logits + (size_t)blockIdx.y * V, from, min(V, from + per), 1);
  if (threadIdx.x == 0) picks[(size_t)blockIdx.y * ARGMAX_PARTS + blockIdx.x] = p;
}
// (one wavefront per row)
__global__ __launch_bounds__(64) void argmax_merge_kernel(const Pick* __restrict__ picks, int* __restrict__ out) {
  Pick p{-INFINITY, ARGMAX_NONE};
  if (threadIdx.x < ARGMAX_PARTS) p = picks[(size_t)blockIdx.x * ARGMAX_PARTS + threadIdx.x];
#pragma unroll
  for (int o = ARGMAX_PARTS / 2; o > 0; o >>= 1) {
    const float ov = __shfl_xor(p.best, o, 64);
    const int oi = __shfl_xor(p.at, o, 64);
    pick_merge(p, ov, oi);
  }
  if (threadIdx.x == 0) out[blockIdx.x] = p.at == ARGMAX_NONE ? 0 : p.at;
}

hipError_t launch_argmax(const float* logits, int* tokens_out, int rows, int V, void* scratch, size_t scratch_per_row, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int vec = V % 4 == 0 && ((uintptr_t)logits & 15) == 0;
  if (vec && V >= ARGMAX_SPLIT_V && rows <= 65535 && scratch_per_row >= ARGMAX_PARTS * sizeof(Pick)) {
    hipLaunchKernelGGL(argmax_part_kernel, dim3(ARGMAX_PARTS, rows), dim3(256), 0, s, logits, (Pick*)scratch, V);
    hipLaunchKernelGGL(argmax_merge_kernel, dim3(rows), dim3(64), 0, s, (const Pick*)scratch, tokens_out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(argmax_kernel, dim3(rows), dim3(1024), 0, s, logits, tokens_out, V, vec);
  return hipGetLastError();
}
