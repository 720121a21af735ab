// Patch embedding + position, the first-layer key score, and the per-token
// cosine similarity against the cached reference (paper §III-B, eq. 3).
//
// Selection must be bit-reproducible, so all three are computed in a fixed
// fp32 order with explicitly rounded operations (no contraction):
//   T[i][d] = fma-chain over k = 0..P-1 of x_i[k] * W_pe[k][d], started at
//             b_pe[d], then one fp32 add of Pos[i][d];
//   key score: x = S(T[i]); mean and variance of x from 64 lane partials
//        (lane j takes d = j, j+64, ... in increasing d: adds for the sum, fma
//        of (x - mean)^2 for the variance) and the halving tree, each / D;
//        rstd = 1 / sqrt(var + eps); n_d = fma((x_d - mean) * rstd, g_d, b_d);
//        key[e] = fma-chain over d of n_d * W_K[d][e] started at b_K[e];
//   cos: lane j of a wave sums the terms d = j, j+64, ... with fma, the 64
//        lane partials are combined by the halving tree (offsets 32..1), then
//        dot / max(sqrt(|a|^2) * sqrt(|b|^2), 1e-8).
// The products are fp32 matrix-core work (P*D fma per token, D*D more for the key).
#include <type_traits>

#include "common.hpp"

namespace incvit {

// The fixed-order product on the matrix cores.  gfx950's fp32 MFMA rounds every
// multiply-add as one fma and takes k in ascending order, so a chain of
// v_mfma_f32_16x16x4_f32 over k is bit for bit the scalar fma chain above
// (checked against host fma chains, denormal results included); it runs at
// twice the vector units' non-packed fp32 rate and needs no LDS.
//
// A wave owns TM x TN tiles of 16 tokens x 16 columns; the product is formed
// transposed (the weights are the MFMA's A operand), so that a lane ends up
// with 4 consecutive columns of one token: 16-byte stores.  One MFMA step takes
// k = 4 s + g from lane group g = lane / 16.
//   * weights: packed so that one 16-byte load per lane (bf16; two for fp32)
//     is a 32-deep chunk of 16 columns, k = 32 c + 4 s + g in element s;
//   * patches: 16-byte loads of 4 consecutive k per lane (64 contiguous bytes
//     per token and half chunk), then a 4 x 4 transposition between the lane
//     groups with v_permlane32_swap / v_permlane16_swap, which puts k = 4 s + g
//     into register s.
// The loads of PF = 4 chunks are in flight (6 to 9 are slower: more lines than
// the first-level cache holds).  The four waves of a workgroup take consecutive
// token tiles of the same columns, so their weight loads meet in that cache.
// Bound by the waves' chains of dependent MFMAs where tiles are few (147 steps
// of 32 clocks at P = 588), by the fp32 matrix rate where they are many.
// Measured, us per launch, against the vector-unit form (LDS-staged, 3 x 2 or
// 4 x 2 outputs per lane) it replaced: 256 x 588 x 1152 21.0 -> 11.8, 3 streams
// of that 30.1 -> 18.6, 1024 x 588 x 1152 40.8 -> 25.6, 2048 x 588 x 1024
// 52.9 -> 31.8, 8192 x 588 x 1024 178 -> 96 (103 TFLOP/s), key projection of
// 546 x 768 x 768 28.7 -> 15.3.

// register j of lane group g <-> register g of lane group j
__device__ __forceinline__ void transpose_groups(uint32_t (&r)[4]) {
  auto s02 = __builtin_amdgcn_permlane32_swap(r[0], r[2], false, false);
  auto s13 = __builtin_amdgcn_permlane32_swap(r[1], r[3], false, false);
  auto s01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
  auto s23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
  r[0] = s01[0];
  r[1] = s01[1];
  r[2] = s23[0];
  r[3] = s23[1];
}

__device__ __forceinline__ void chunk_weights(float* f, const V8<uint16_t>& v) {
  const uint32_t q[4] = {v.v.x, v.v.y, v.v.z, v.v.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(q[e] << 16);
    f[2 * e + 1] = __uint_as_float(q[e] & 0xffff0000u);
  }
}
__device__ __forceinline__ void chunk_weights(float* f, const V8<float>& v) {
  f[0] = v.a.x; f[1] = v.a.y; f[2] = v.a.z; f[3] = v.a.w;
  f[4] = v.b.x; f[5] = v.b.y; f[6] = v.b.z; f[7] = v.b.w;
}

template <class T, int TM, int TN>
__device__ __forceinline__ void embed_body(const EmbedArgs& a) {
  constexpr int PF = 4;            // chunks in flight
  constexpr int TT = 4 * TM * 16;  // tokens per workgroup
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, n = lane & 15;
  // Workgroups are dealt to the 8 XCDs round robin by linear launch index, and
  // each XCD has its own L2.  Renumber them XCD-major (a bijection) and take
  // (stream, column block, token group) from the new number, so that the
  // workgroups of one column block sit on one XCD (at most two): its weights
  // come from HBM once rather than once per XCD.
  const int N = a.N, P = a.P, D = a.D;
  const int ntg = (N + TT - 1) / TT, ncb = D / (16 * TN);
  const int total = ntg * ncb * a.B;
  const int i = blockIdx.x;
  const int x = i % 8, q = total / 8, rem = total % 8;
  const int pos = x * q + min(x, rem) + i / 8;
  const int v = pos / (ncb * ntg), cb = (pos / ntg) % ncb, tg = pos % ntg;

  if (tg == 0 && cb == 0 && a.ident_idx) {
    for (int k = tid; k < N; k += 256) a.ident_idx[v * N + k] = k;
    if (tid == 0) a.ident_count[v] = N;
  }
  const int tok0 = tg * TT + w * TM * 16;  // first token of this wave
  if (tok0 >= N) return;                   // uniform; no barriers below

  const int nc = (P + 31) / 32;
  const Rsrc rx = make_rsrc(a.patches + (size_t)v * N * P, (uint32_t)((size_t)N * P * 4));
  const size_t wblk = (size_t)nc * kChunkElems;  // elements of one 16-column block
  const T* wbase = static_cast<const T*>(a.w_pe) + (size_t)cb * TN * wblk;
  const Rsrc rw = make_rsrc(wbase, (uint32_t)(TN * wblk * sizeof(T)));
  uint32_t xoff[TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) xoff[t] = (uint32_t)((min(tok0 + 16 * t + n, N - 1) * P + 4 * g) * 4);
  const uint32_t woff = (uint32_t)(lane * 8 * sizeof(T));

  struct Chunk {
    float4 x[TM][2];
    V8<T> w[TN];
  };
  auto fetch = [&](Chunk& ch, int c) {
#pragma unroll
    for (int b = 0; b < TN; ++b) ch.w[b].bload(rw, woff, (uint32_t)((b * wblk + (size_t)c * kChunkElems) * sizeof(T)));
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) ch.x[t][h] = bload16f(rx, xoff[t], (uint32_t)(32 * c + 16 * h) * 4);
  };
  f32x4_t acc[TM][TN];
  float4 posv[TM][TN];
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int d = (cb * TN + b) * 16 + 4 * g;
    const float4 bias = *reinterpret_cast<const float4*>(a.b_pe + d);
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      acc[t][b] = f32x4_t{bias.x, bias.y, bias.z, bias.w};
      const int tok = min(tok0 + 16 * t + n, N - 1);
      posv[t][b] = a.pos ? *reinterpret_cast<const float4*>(a.pos + (size_t)tok * D + d) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
  }
  // the 8 steps of a chunk (steps: how many of them hold k < P; values past P
  // within a step are zeroed on both sides)
  auto compute = [&](const Chunk& ch, auto last, int c) {
    constexpr bool LAST = decltype(last)::value;
    float wv[TN][8];
#pragma unroll
    for (int b = 0; b < TN; ++b) chunk_weights(wv[b], ch.w[b]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k0 = 32 * c + 16 * h;
      uint32_t xr[TM][4];
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        const float xs[4] = {ch.x[t][h].x, ch.x[t][h].y, ch.x[t][h].z, ch.x[t][h].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) xr[t][j] = !LAST || k0 + 4 * g + j < P ? __float_as_uint(xs[j]) : 0u;
        transpose_groups(xr[t]);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (LAST && k0 + 4 * s >= P) continue;  // uniform
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
          for (int b = 0; b < TN; ++b)
            acc[t][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[b][4 * h + s], __uint_as_float(xr[t][s]), acc[t][b], 0, 0, 0);
      }
    }
  };
  // chunk c sits in register slot c % PF; a slot is refilled right after its use
  Chunk ch[PF];
#pragma unroll
  for (int p = 0; p < PF; ++p) fetch(ch[p], p);  // past the end: zeros or unused data of the next row
  const int full = P / 32;  // chunks without a tail
  int c = 0;
  for (; c + PF <= full; c += PF) {
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      compute(ch[p], std::false_type{}, c + p);
      fetch(ch[p], c + p + PF);
    }
  }
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (c + p < nc) compute(ch[p], std::true_type{}, c + p);  // uniform

#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int tok = tok0 + 16 * t + n;
    if (tok >= N) continue;
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      float4 o = make_float4(acc[t][b][0], acc[t][b][1], acc[t][b][2], acc[t][b][3]);
      if (a.pos)
        o = make_float4(__fadd_rn(o.x, posv[t][b].x), __fadd_rn(o.y, posv[t][b].y), __fadd_rn(o.z, posv[t][b].z),
                        __fadd_rn(o.w, posv[t][b].w));
      *reinterpret_cast<float4*>(a.t0 + ((size_t)v * N + tok) * D + (cb * TN + b) * 16 + 4 * g) = o;
    }
  }
}

template <class T, int TM, int TN>
__global__ __launch_bounds__(256) void embed_kernel(EmbedArgs a) {
  embed_body<T, TM, TN>(a);
}

// The key projection of the key score: the same fixed-order product with
// x = LayerNorm rows, K = D, W = W_K of layer 0, no position term.
template <class T, int TM, int TN>
__global__ __launch_bounds__(256) void keyproj_kernel(EmbedArgs a) {
  embed_body<T, TM, TN>(a);
}

// Correctly rounded fp32 square root.  HIP's __fsqrt_rn is the bare hardware
// square root (about 1 ulp) unless OCML's rounded operations are enabled;
// __builtin_sqrtf compiles to the hardware estimate plus the fma correction
// that rounds it correctly (the fp32 divide is correctly rounded by default).
__device__ __forceinline__ float sqrt_rn(float x) { return __builtin_sqrtf(x); }

// Sum of the 64 lane values by the halving tree; lane 0's value is the
// result, broadcast to the wave.
__device__ __forceinline__ float tree64(float p) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) p = __fadd_rn(p, __shfl_down(p, off, 64));
  return __shfl(p, 0, 64);
}

// One wave per token: n = LayerNorm 1 of layer 0 on S(T0[token]), fixed order.
template <class T>
__global__ __launch_bounds__(256) void keyln_kernel(KeyLnArgs a) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = blockIdx.x * 4 + w;
  if (row >= a.rows) return;
  const int D = a.D;
  const float* x = a.t0 + (size_t)row * D;
  constexpr int kPer = kMaxDim / 64;
  float xv[kPer], g[kPer], b[kPer];
  // unconditional loads (clamped index), all issued before any is used; the
  // values past D are never used
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int d = min(lane + 64 * j, D - 1);
    xv[j] = x[d];
    g[j] = a.ln_g[d];
    b[j] = a.ln_b[d];
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) xv[j] = Elem<T>::rnd(xv[j]);
  float p = 0.0f;
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (lane + 64 * j < D) p = __fadd_rn(p, xv[j]);
  const float mean = __fdiv_rn(tree64(p), (float)D);
  float q = 0.0f;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    xv[j] = __fsub_rn(xv[j], mean);
    if (lane + 64 * j < D) q = __fmaf_rn(xv[j], xv[j], q);
  }
  const float var = __fdiv_rn(tree64(q), (float)D);
  const float rstd = __fdiv_rn(1.0f, sqrt_rn(__fadd_rn(var, a.eps)));
  float* out = a.out + (size_t)row * D;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int d = lane + 64 * j;
    if (d < D) out[d] = __fmaf_rn(__fmul_rn(xv[j], rstd), g[j], b[j]);
  }
}

// One wave per token: cos(T0[v][i], ref[v][i]); the wave's loads go out in one batch.
__global__ __launch_bounds__(256) void sim_kernel(SimArgs a) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gt = blockIdx.x * 4 + w;
  if (gt >= a.B * a.N) return;
  const int v = gt / a.N, tok = gt - v * a.N;
  const float* x = a.t0 + (size_t)gt * a.D;
  const float* y = reinterpret_cast<const float*>(a.caches.p[v] + a.ref_off) + (size_t)tok * a.D;
  constexpr int kPer = kMaxDim / 64;
  float xv[kPer], yv[kPer];
  // unconditional loads (clamped index), all issued before any is used; the
  // values past D are never used
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int d = min(lane + 64 * j, a.D - 1);
    xv[j] = x[d];
    yv[j] = y[d];
  }
  float pd = 0.0f, pa = 0.0f, pb = 0.0f;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {  // d = lane + 64 j in increasing d; entries past D are skipped
    if (lane + 64 * j < a.D) {
      pd = __fmaf_rn(xv[j], yv[j], pd);
      pa = __fmaf_rn(xv[j], xv[j], pa);
      pb = __fmaf_rn(yv[j], yv[j], pb);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    pd = __fadd_rn(pd, __shfl_down(pd, off, 64));
    pa = __fadd_rn(pa, __shfl_down(pa, off, 64));
    pb = __fadd_rn(pb, __shfl_down(pb, off, 64));
  }
  if (lane == 0) {
    const float denom = __fmul_rn(sqrt_rn(pa), sqrt_rn(pb));
    a.sim[gt] = __fdiv_rn(pd, fmaxf(denom, 1e-8f));
  }
}

// Tiles per wave, by the number of 16 x 16 output tiles (the chip has 1024
// SIMDs): one while they are about two per SIMD or fewer, so that every SIMD
// has a chain to run (1152 tiles 11.8 us against 13.5 with 1 x 2; 2304 tiles
// 14.8 against 16.7); then 1 x 2, which reads each token row for 32 columns
// (3456 tiles 18.6 against 20.2); and 2 x 4 from 16 tiles per SIMD on, where
// operand reads set the pace (32768 tiles 96 against 103; 8192 tiles equal).
template <class T, bool KEY>
hipError_t launch_product(const EmbedArgs& a, hipStream_t s) {
  auto go = [&](auto kernel, int tm, int tn) {
    const int tt = 64 * tm;
    return launch_k(kernel, dim3((a.N + tt - 1) / tt * (a.D / (16 * tn)) * a.B), dim3(256), 0, s, a);
  };
  const long tiles = (long)a.B * ((a.N + 15) / 16) * (a.D / 16);
  if (tiles <= 2560) return KEY ? go(keyproj_kernel<T, 1, 1>, 1, 1) : go(embed_kernel<T, 1, 1>, 1, 1);
  if (tiles < 16384 || a.D % 64) return KEY ? go(keyproj_kernel<T, 1, 2>, 1, 2) : go(embed_kernel<T, 1, 2>, 1, 2);
  return KEY ? go(keyproj_kernel<T, 2, 4>, 2, 4) : go(embed_kernel<T, 2, 4>, 2, 4);
}

hipError_t launch_embed(const EmbedArgs& a, hipStream_t s) {
  return a.dtype ? launch_product<uint16_t, false>(a, s) : launch_product<float, false>(a, s);
}

hipError_t launch_keyproj(const EmbedArgs& a, hipStream_t s) {
  return a.dtype ? launch_product<uint16_t, true>(a, s) : launch_product<float, true>(a, s);
}

hipError_t launch_keyln(const KeyLnArgs& a, hipStream_t s) {
  dim3 grid((a.rows + 3) / 4);
  if (a.dtype) return launch_k(keyln_kernel<uint16_t>, grid, dim3(256), 0, s, a);
  return launch_k(keyln_kernel<float>, grid, dim3(256), 0, s, a);
}

hipError_t launch_sim(const SimArgs& a, hipStream_t s) {
  dim3 grid((a.B * a.N + 3) / 4);
  (void)launch_k(sim_kernel, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace incvit
