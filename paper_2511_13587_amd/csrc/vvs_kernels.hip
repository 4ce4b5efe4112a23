// Element-wise / reduction kernels of the verify pass, the fp32 (reference-shape) GEMM and attention
// kernels, weight repacking, KV commit, and the launch sequence of one transformer forward.
// The bf16 GEMM and attention kernels (MFMA) live in vvs_mfma.hip; the acceptance stage in
// vvs_accept.hip.
#include "vvs_device.h"

#include <stdlib.h>
#include <algorithm>

namespace vvs {

// ------------------------------------------------------------------------------------------------ utilities
__global__ void k_fill_zero(uint4* p, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const uint4 z = make_uint4(0, 0, 0, 0);
  for (; i < n16; i += stride) p[i] = z;
}

void launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  size_t n16 = bytes / 16;
  if (!n16) return;
  int blocks = (int)std::min<size_t>((n16 + 255) / 256, 256 * 32);
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, s, (uint4*)p, n16);
}

__global__ void k_copy_bytes(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) dst[i] = src[i];
}

void launch_copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t s) {
  size_t n16 = bytes / 16;
  if (!n16) return;
  int blocks = (int)std::min<size_t>((n16 + 255) / 256, 256 * 32);
  hipLaunchKernelGGL(k_copy_bytes, dim3(blocks), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, n16);
}

// out[n][k] = in[k][col0 + n]   (in: [K][ld])
template <typename T>
__global__ void k_transpose(const T* __restrict__ in, T* __restrict__ out, int K, int N, int ld, int col0) {
  __shared__ T tile[32][33];
  const int n0 = blockIdx.x * 32, k0 = blockIdx.y * 32;
  for (int i = threadIdx.y; i < 32; i += 8) {
    int k = k0 + i, n = n0 + threadIdx.x;
    if (k < K && n < N) tile[i][threadIdx.x] = in[(size_t)k * ld + col0 + n];
  }
  __syncthreads();
  for (int i = threadIdx.y; i < 32; i += 8) {
    int n = n0 + i, k = k0 + threadIdx.x;
    if (k < K && n < N) out[(size_t)n * K + k] = tile[threadIdx.x][i];
  }
}

// bf16 weights: out = packed fragment order of W^T, i.e. rows = output features n, contraction = k;
// in[k][col0 + n].  One thread per 16-byte chunk; the 32 lanes of a half-block read 32 consecutive n.
// Row block nb of the source lands in row block nb * nb_stride + nb_off of the destination (gate and
// up projections are interleaved block by block so that one GEMM tile holds both for the same units).
// The weights are copied bit for bit: the packed operand holds exactly the bf16 values the caller gave.
__global__ void k_pack_w(const bf16_t* __restrict__ in, uint4* __restrict__ out, int K, int N, int ld, int col0, int nb_stride,
                         int nb_off) {
  const size_t chunk = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t total = (size_t)(N >> 5) * (K >> 4) * 64;
  if (chunk >= total) return;
  const int lane = (int)(chunk & 63);
  const size_t blk = chunk >> 6;
  const int kb = (int)(blk % (K >> 4)), nb = (int)(blk / (K >> 4));
  const int n = nb * 32 + (lane & 31), k0 = kb * 16 + (lane >> 5) * 8;
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t lo = in[(size_t)(k0 + 2 * i) * ld + col0 + n], hi = in[(size_t)(k0 + 2 * i + 1) * ld + col0 + n];
    w[i] = lo | (hi << 16);
  }
  out[(((size_t)nb * nb_stride + nb_off) * (K >> 4) + kb) * 64 + lane] = make_uint4(w[0], w[1], w[2], w[3]);
}

// bf16 activations, row-major [M][K] -> packed fragment order (rows beyond M are zero)
__global__ void k_pack_a(const bf16_t* __restrict__ in, uint4* __restrict__ out, int M, int K) {
  const size_t chunk = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t total = (size_t)((M + 31) >> 5) * (K >> 4) * 64;
  if (chunk >= total) return;
  const int lane = (int)(chunk & 63);
  const size_t blk = chunk >> 6;
  const int kb = (int)(blk % (K >> 4)), mb = (int)(blk / (K >> 4));
  const int m = mb * 32 + (lane & 31), k0 = kb * 16 + (lane >> 5) * 8;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (m < M) v = *(const uint4*)(in + (size_t)m * K + k0);
  out[chunk] = v;
}

template <typename T>
static void transpose_into(const void* in, void* out, int K, int N, int ld, int col0, hipStream_t s, int nb_stride = 1, int nb_off = 0) {
  if (sizeof(T) == 2) {
    const size_t total = (size_t)(N >> 5) * (K >> 4) * 64;
    hipLaunchKernelGGL(k_pack_w, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (const bf16_t*)in, (uint4*)out, K, N, ld, col0,
                       nb_stride, nb_off);
    return;
  }
  dim3 grid((N + 31) / 32, (K + 31) / 32);
  hipLaunchKernelGGL(k_transpose<T>, grid, dim3(32, 8), 0, s, (const T*)in, (T*)out, K, N, ld, col0);
}

template <typename T>
__global__ void k_copy(const T* __restrict__ in, T* __restrict__ out, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i < n; i += (size_t)gridDim.x * blockDim.x) out[i] = in[i];
}
template <typename T>
__global__ void k_to_float(const T* __restrict__ in, float* __restrict__ out, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i < n; i += (size_t)gridDim.x * blockDim.x) out[i] = ld(in + i);
}

template <typename T>
static void pack_weights_t(Ctx* c, const void* const* t, hipStream_t s) {
  const int d = c->d, F = c->F;
  auto copy = [&](const void* in, size_t off, size_t n) {
    int blocks = (int)std::min<size_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_copy<T>, dim3(blocks), dim3(256), 0, s, (const T*)in, (T*)(c->pw + off), n);
  };
  auto gain = [&](const void* in, size_t off) {
    hipLaunchKernelGGL(k_to_float<T>, dim3((d + 255) / 256), dim3(256), 0, s, (const T*)in, (float*)(c->pw + off), (size_t)d);
  };
  copy(t[0], c->p.embed, (size_t)c->V * d);
  if (t[1]) copy(t[1], c->p.prefix_embed, (size_t)(c->cfg.n_classes + 1) * d);
  for (int l = 0; l < c->L; ++l) {
    const void* const* w = t + 2 + 9 * l;
    size_t base = c->p.layer0 + c->p.layer_stride * l;
    gain(w[0], base + c->p.g1);
    char* qkv = c->pw + base + c->p.wqkv;
    for (int i = 0; i < 3; ++i) transpose_into<T>(w[1 + i], qkv + (size_t)i * d * d * sizeof(T), d, d, d, 0, s);
    transpose_into<T>(w[4], c->pw + base + c->p.wo, d, d, d, 0, s);
    gain(w[5], base + c->p.g2);
    char* gu = c->pw + base + c->p.wgu;
    if (sizeof(T) == 2) {            // bf16: gate / up interleaved in blocks of 32 output features
      transpose_into<T>(w[6], gu, d, F, F, 0, s, 2, 0);
      transpose_into<T>(w[7], gu, d, F, F, 0, s, 2, 1);
    } else {
      transpose_into<T>(w[6], gu, d, F, F, 0, s);
      transpose_into<T>(w[7], gu + (size_t)F * d * sizeof(T), d, F, F, 0, s);
    }
    transpose_into<T>(w[8], c->pw + base + c->p.wd, F, d, d, 0, s);
  }
  const void* const* tail = t + 2 + 9 * c->L;
  gain(tail[0], c->p.gf);
  transpose_into<T>(tail[1], c->pw + c->p.wout, d, c->veff, c->V, c->lo, s);
  if (c->cfg.draft_input) transpose_into<T>(tail[2], c->pw + c->p.fc, 2 * d, d, d, 0, s);
}

void launch_pack_weights(Ctx* c, const void* const* tensors, hipStream_t s) {
  if (c->cfg.dtype == VVS_BF16) pack_weights_t<bf16_t>(c, tensors, s);
  else pack_weights_t<float>(c, tensors, s);
}

// ------------------------------------------------------------------------------------------------ embedding
struct EmbedArgs {
  int T, d, V, mode;                 // mode 0: verify (token table), 1: prefill chunk
  const int32_t* tokens_bt;          // [B][T]
  const void* pc; const void* pu;    // prefix inputs
  int prefix_kind, n_classes, P, chunk_start, n_forced;
  const int32_t* forced;
};

template <typename T>
__device__ __forceinline__ const T* embed_source(const T* __restrict__ embed, const T* __restrict__ prefix_tab, const EmbedArgs& a, int m) {
  const int r = m / a.T, t = m % a.T, b = r >> 1;
  const T* src;
  if (a.mode == 0) {
    int tok = min(max(a.tokens_bt[b * a.T + t], 0), a.V - 1);
    src = embed + (size_t)tok * a.d;
  } else {
    int slot = a.chunk_start + t;
    if (slot < a.P) {
      if (a.prefix_kind == VVS_PREFIX_CLASS) {
        int id;
        if (r & 1) id = a.pu ? ((const int32_t*)a.pu)[b * a.P + slot] : a.n_classes;
        else id = ((const int32_t*)a.pc)[b * a.P + slot];
        id = min(max(id, 0), a.n_classes);
        src = prefix_tab + (size_t)id * a.d;
      } else {
        src = (r & 1) ? (const T*)a.pu + (size_t)slot * a.d : (const T*)a.pc + ((size_t)b * a.P + slot) * a.d;
      }
    } else {
      int tok = min(max(a.forced[b * a.n_forced + slot - a.P], 0), a.V - 1);
      src = embed + (size_t)tok * a.d;
    }
  }
  return src;
}

template <typename T>
__global__ void k_embed(float* __restrict__ x, const T* __restrict__ embed, const T* __restrict__ prefix_tab, EmbedArgs a) {
  const int m = blockIdx.x;
  const T* src = embed_source(embed, prefix_tab, a, m);
  for (int i = threadIdx.x; i < a.d; i += blockDim.x) x[(size_t)m * a.d + i] = ld(src + i);
}

// Embedding for the path without separate normalisation kernels: x (fp32), bf16(x * g) in packed operand
// order (g = gain of the norm that follows), and the row's sum of squares (slab 0 holds the whole sum, the
// other slabs 0).
__global__ __launch_bounds__(256) void k_embed_packed(float* __restrict__ x, bf16_t* __restrict__ xb, float* __restrict__ ss, int NS,
                                                      const bf16_t* __restrict__ embed, const bf16_t* __restrict__ prefix_tab,
                                                      const float* __restrict__ g, EmbedArgs a, int pad_T, int pad) {
  __shared__ float red[16];
  const int m = blockIdx.x;
  const int mp = pad_T > 0 ? (m / pad_T) * pad + m % pad_T : m;   // row of the packed operand (row-padded layout: pad rows per pad_T tokens)
  const bf16_t* src = embed_source(embed, prefix_tab, a, m);
  float sq = 0.f;
  for (int k0 = threadIdx.x * 8; k0 < a.d; k0 += 256 * 8) {
    const uint4 raw = *(const uint4*)(src + k0);
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
    float v[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[2 * i] = bf2f((bf16_t)(w[i] & 0xFFFF)); v[2 * i + 1] = bf2f((bf16_t)(w[i] >> 16)); }
    store8(x, m, k0, a.d, v);
    const float4 ga = *(const float4*)(g + k0), gb = *(const float4*)(g + k0 + 4);
    const float hv[8] = {v[0] * ga.x, v[1] * ga.y, v[2] * ga.z, v[3] * ga.w, v[4] * gb.x, v[5] * gb.y, v[6] * gb.z, v[7] * gb.w};
    store8(xb, mp, k0, a.d, hv);
#pragma unroll
    for (int i = 0; i < 8; ++i) sq += v[i] * v[i];
  }
  sq = block_sum(sq, red);
  if (threadIdx.x < NS) ss[(size_t)m * NS + threadIdx.x] = threadIdx.x == 0 ? sq : 0.f;
}

// Rows (i * stride + off) of x, times the gain g -> packed bf16 rows i, with their sums of squares (for the lm_head of a prefill)
__global__ __launch_bounds__(256) void k_gather_rows(const float* __restrict__ x, const float* __restrict__ ss, const float* __restrict__ g,
                                                     bf16_t* __restrict__ xb2, float* __restrict__ ss2, int d, int NS, int stride, int off) {
  const int i = blockIdx.x;
  const size_t m = (size_t)i * stride + off;
  for (int k0 = threadIdx.x * 8; k0 < d; k0 += 256 * 8) {
    const float4 a = *(const float4*)(x + m * d + k0), b = *(const float4*)(x + m * d + k0 + 4);
    const float4 ga = *(const float4*)(g + k0), gb = *(const float4*)(g + k0 + 4);
    const float v[8] = {a.x * ga.x, a.y * ga.y, a.z * ga.z, a.w * ga.w, b.x * gb.x, b.y * gb.y, b.z * gb.z, b.w * gb.w};
    store8(xb2, i, k0, d, v);
  }
  if (threadIdx.x < NS) ss2[(size_t)i * NS + threadIdx.x] = ss[m * NS + threadIdx.x];
}

__global__ void k_build_tokens(int32_t* __restrict__ tokens, const int32_t* __restrict__ pending, const int32_t* __restrict__ draft,
                               int B, int T) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= B * T) return;
  int b = i / T, j = i % T;
  tokens[i] = j == 0 ? pending[b] : draft[b * (T - 1) + j - 1];
}

void launch_build_tokens(Ctx* c, int T, const int32_t* d_draft, hipStream_t s) {
  Timed timed(c, VVS_K_ELEMENTWISE, s);
  int n = c->B * T;
  const int32_t* pending = (const int32_t*)(c->ws + c->w.state) + 2 * c->B;
  hipLaunchKernelGGL(k_build_tokens, dim3((n + 255) / 256), dim3(256), 0, s, (int32_t*)(c->ws + c->w.tokens), pending, d_draft,
                     c->B, T);
}

// ------------------------------------------------------------------------------------------------ residual add + RMSNorm
// Output row i reads x row (i * in_stride + in_off): x_row += sum of GEMM partials (if any), then
// h_row = x_row / sqrt(mean(x_row^2) + eps) * g, rounded to the operand type.
template <typename T, int NCH, int NT>
__global__ __launch_bounds__(NT) void k_add_rmsnorm(float* __restrict__ x, const float* __restrict__ partial, int splits,
                                                     size_t split_stride, int d, const float* __restrict__ g, float eps,
                                                     T* __restrict__ h, int in_stride, int in_off) {
  // each of the NT threads owns NCH chunks of 8 consecutive values of the row (d <= NCH * NT * 8) and keeps them in
  // registers between the sum of squares and the scaling; one chunk per thread where the row allows it, so that
  // everything a row needs is requested in one round trip to memory
  __shared__ float red[16];
  const size_t row = (size_t)blockIdx.x * in_stride + in_off;
  float* xr = x + row * d;
  float xv[NCH][8];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int k0 = (threadIdx.x + NT * j) * 8;
    if (k0 < d) {
      const float4 a = *(const float4*)(xr + k0), b = *(const float4*)(xr + k0 + 4);
      float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      if (splits) {
        // all partial sums of the chunk are requested before the first is added (the planner makes at most 8 splits): one
        // round trip to memory per chunk instead of one per split; added in the order of the splits
        constexpr int kMaxSplits = 8;
        float4 pa[kMaxSplits], pb[kMaxSplits];
#pragma unroll
        for (int s = 0; s < kMaxSplits; ++s) {
          if (s < splits) {
            const float* pr = partial + s * split_stride + row * d + k0;
            pa[s] = *(const float4*)pr;
            pb[s] = *(const float4*)(pr + 4);
          }
        }
#pragma unroll
        for (int s = 0; s < kMaxSplits; ++s) {
          if (s < splits) {
            v[0] += pa[s].x; v[1] += pa[s].y; v[2] += pa[s].z; v[3] += pa[s].w;
            v[4] += pb[s].x; v[5] += pb[s].y; v[6] += pb[s].z; v[7] += pb[s].w;
          }
        }
        for (int s = kMaxSplits; s < splits; ++s) {          // not reached with the planner's limit
          const float* pr = partial + s * split_stride + row * d + k0;
          const float4 qa = *(const float4*)pr, qb = *(const float4*)(pr + 4);
          v[0] += qa.x; v[1] += qa.y; v[2] += qa.z; v[3] += qa.w; v[4] += qb.x; v[5] += qb.y; v[6] += qb.z; v[7] += qb.w;
        }
        *(float4*)(xr + k0) = make_float4(v[0], v[1], v[2], v[3]);
        *(float4*)(xr + k0 + 4) = make_float4(v[4], v[5], v[6], v[7]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) { xv[j][i] = v[i]; ss += v[i] * v[i]; }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) xv[j][i] = 0.f;
    }
  }
  ss = block_sum(ss, red);
  const float scale = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int k0 = (threadIdx.x + NT * j) * 8;
    if (k0 < d) {
      float gv[8] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
      if (g) {
        const float4 ga = *(const float4*)(g + k0), gb = *(const float4*)(g + k0 + 4);
        gv[0] = ga.x; gv[1] = ga.y; gv[2] = ga.z; gv[3] = ga.w; gv[4] = gb.x; gv[5] = gb.y; gv[6] = gb.z; gv[7] = gb.w;
      }
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = xv[j][i] * scale * gv[i];
      store8(h, (int)blockIdx.x, k0, d, v);
    }
  }
}

template <typename T>
static void launch_add_rmsnorm(int rows, float* x, const float* partial, int splits, size_t split_stride, int d, const float* g, float eps,
                               T* h, int in_stride, int in_off, hipStream_t s) {
  if (d <= 2048)
    hipLaunchKernelGGL((k_add_rmsnorm<T, 1, 256>), dim3(rows), dim3(256), 0, s, x, partial, splits, split_stride, d, g, eps, h, in_stride, in_off);
  else if (d <= 4096)
    hipLaunchKernelGGL((k_add_rmsnorm<T, 1, 512>), dim3(rows), dim3(512), 0, s, x, partial, splits, split_stride, d, g, eps, h, in_stride, in_off);
  else
    hipLaunchKernelGGL((k_add_rmsnorm<T, 8, 256>), dim3(rows), dim3(256), 0, s, x, partial, splits, split_stride, d, g, eps, h, in_stride, in_off);
}

// ------------------------------------------------------------------------------------------------ RoPE + KV write
template <typename T>
__global__ void k_rope_kv(const float* __restrict__ qkv, int splits, size_t split_stride, T* __restrict__ q, T* __restrict__ kc,
                          T* __restrict__ vc, const float* __restrict__ rope_tab, TreeDesc tree, PosDesc pos, int T_, int d,
                          int dh, size_t row_stride, size_t head_stride, int S_cap, int rope_pos) {
  const int m = blockIdx.x, r = m / T_, t = m % T_;
  int slot, img;
  token_pos(pos, tree, r, t, &slot, &img);
  const int half = dh >> 1, np = dh >> 2;
  int gr = 0, gc = 0;
  if (img >= 0) { gr = min(img / pos.grid_w, rope_pos - 1); gc = img % pos.grid_w; }
  const bool in_cache = slot >= 0 && slot < S_cap;
  const size_t n3 = (size_t)3 * d;
  for (int i = blockIdx.y * blockDim.x + threadIdx.x; i < (d >> 1); i += gridDim.y * blockDim.x) {   // one pair per thread
    const int e0 = 2 * i, hd = e0 / dh, e = e0 % dh;
    const int seg = e / half, ip = (e % half) >> 1;
    float cs = 1.f, sn = 0.f;
    if (img >= 0) {
      const int pv = seg ? gc : gr;
      cs = rope_tab[((size_t)pv * np + ip) * 2];
      sn = rope_tab[((size_t)pv * np + ip) * 2 + 1];
    }
    float v[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < splits; ++s) {
      const float* row = qkv + s * split_stride + (size_t)m * n3;
      v[0] += row[e0]; v[1] += row[e0 + 1];
      v[2] += row[d + e0]; v[3] += row[d + e0 + 1];
      v[4] += row[2 * d + e0]; v[5] += row[2 * d + e0 + 1];
    }
    st(q + (size_t)m * d + e0, v[0] * cs - v[1] * sn);
    st(q + (size_t)m * d + e0 + 1, v[0] * sn + v[1] * cs);
    if (in_cache) {
      const size_t hb = (size_t)r * row_stride + (size_t)hd * head_stride;
      st(kc + hb + k_index(slot, e, dh), v[2] * cs - v[3] * sn);
      st(kc + hb + k_index(slot, e + 1, dh), v[2] * sn + v[3] * cs);
      st(vc + hb + v_index(slot, e, dh), v[4]);
      st(vc + hb + v_index(slot, e + 1, dh), v[5]);
    }
  }
}

// ------------------------------------------------------------------------------------------------ attention, one query per workgroup
// Bound by chains of loads: a thread takes whole keys for the scores (16-byte pieces of the key, all requested before the
// first is used), and the P V sum is dealt to 256 / dh groups of dh threads by chunks of 8 keys - contiguous in the cache's V
// order - whose partial sums are added in a fixed order.  One group over all keys, one element at a time, took 11.9 us at 40
// keys and head size 32; 5.8 us.
__global__ __launch_bounds__(256) void k_attn_simple(const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
                              float* __restrict__ out, TreeDesc tree, PosDesc pos, int T_, int d, int dh, size_t row_stride, size_t head_stride, int S_cap) {
  extern __shared__ float sc[];          // [S_cap] scores, then 16 floats for reductions
  __shared__ float part[256];            // [group][dim]
  float* red = sc + S_cap;
  const int t = blockIdx.x, hd = blockIdx.y, r = blockIdx.z, m = r * T_ + t;
  const int S = pos.kv_len ? pos.kv_len[r >> 1] : pos.kv_base;
  const int n = min(S + tree.first + T_, S_cap);
  const uint64_t mask = tree.anc[tree.first + t];
  const float* qv = q + (size_t)m * d + (size_t)hd * dh;
  const float* kb = kc + (size_t)r * row_stride + (size_t)hd * head_stride;
  const float* vb = vc + (size_t)r * row_stride + (size_t)hd * head_stride;
  const float scale = 1.0f / sqrtf((float)dh);
  float mx = -INFINITY;
  for (int k = threadIdx.x; k < n; k += 256) {
    bool vis = k < S || ((mask >> (k - S)) & 1ull);
    float sv = -INFINITY;
    if (vis) {
      float dot = 0.f;
#pragma unroll 8
      for (int e = 0; e < dh; e += 4) {    // the head size is a multiple of 4, and 4 dims of a key are contiguous in either K order
        const float4 a = *(const float4*)(qv + e), kk = *(const float4*)(kb + k_index(k, e, dh));
        dot += (a.x * kk.x + a.y * kk.y) + (a.z * kk.z + a.w * kk.w);
      }
      sv = dot * scale;
    }
    sc[k] = sv;
    mx = fmaxf(mx, sv);
  }
  mx = block_max(mx, red);
  float sum = 0.f;
  for (int k = threadIdx.x; k < n; k += 256) {
    float e = sc[k] == -INFINITY ? 0.f : expf(sc[k] - mx);
    sc[k] = e;
    sum += e;
  }
  sum = block_sum(sum, red);               // its barriers also publish the weights
  const int ng = 256 / dh, g = threadIdx.x / dh, e = threadIdx.x % dh;   // head sizes up to 256
  float o = 0.f;
  if (g < ng)
    for (int k0 = 8 * g; k0 < n; k0 += 8 * ng) {
      const float4* vp = (const float4*)(vb + v_index(k0, e, dh));       // 8 consecutive slots of a dim; the region holds whole steps of 32
      const float4 v0 = vp[0], v1 = vp[1];
      const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) o += k0 + i < n ? sc[k0 + i] * v[i] : 0.f;   // slots from n on hold anything
    }
  part[threadIdx.x] = o;                   // [g][e]
  __syncthreads();
  if (g == 0) {
    for (int j = 1; j < ng; ++j) o += part[j * dh + e];
    out[(size_t)m * d + (size_t)hd * dh + e] = o / sum;
  }
}

// ------------------------------------------------------------------------------------------------ SwiGLU
template <typename T>
__global__ void k_swiglu(const float* __restrict__ gu, int splits, size_t split_stride, T* __restrict__ act, int M, int F,
                         int interleaved) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;      // one thread per 8 consecutive f
  const int per_row = F >> 3;
  if (i >= (size_t)M * per_row) return;
  const int m = (int)(i / per_row), f0 = (int)(i % per_row) * 8;
  float g[8], u[8], v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) g[k] = u[k] = 0.f;
  for (int s = 0; s < splits; ++s) {
    const float* row = gu + s * split_stride + (size_t)m * 2 * F;
    // column of gate unit f: f (then up at F + f), or interleaved in blocks of 32: (f/32)*64 + f%32 (up 32 further)
    const int gc = interleaved ? (f0 >> 5) * 64 + (f0 & 31) : f0, uc = interleaved ? gc + 32 : F + f0;
#pragma unroll
    for (int k = 0; k < 8; ++k) { g[k] += row[gc + k]; u[k] += row[uc + k]; }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = g[k] / (1.0f + expf(-g[k])) * u[k];
  store8(act, m, f0, F, v);
}

// ------------------------------------------------------------------------------------------------ GEMM, one wave per output column
// C[m][n] = sum_k A[m][k] * W[n][k] in fp32; a wave owns one column for 8 rows of A, its lanes stride over k.  The matrices of
// this path are small and a launch lasts as long as its chain of loads, so everything is asked for before the first product:
// rows past M repeat the last one instead of being skipped behind a branch each, VEC lanes take 16 bytes at a time and 2 x 64
// such pieces (K = 512) are under way at once.  Launch of 128 columns and 10 rows, K 128 and 344 on average: 11.4 us with
// 4-byte loads behind the row tests, 3.5 us so.  !VEC: a K that is not a multiple of 4, or operands not on 16 bytes.
template <bool VEC>
__global__ __launch_bounds__(256) void k_gemm_simple(const float* __restrict__ A, const float* __restrict__ W, float* __restrict__ C, int M, int N, int K, RowMap out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = blockIdx.x * 4 + wave, m0 = blockIdx.y * 8;
  if (n >= N) return;
  const float* w = W + (size_t)n * K;
  const float* a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = A + (size_t)min(m0 + i, M - 1) * K;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  if constexpr (VEC) {
    const int K4 = K >> 2;
    for (int k0 = 0; k0 < K4; k0 += 128) {
      float4 wv[2], av[2][8];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = k0 + 64 * u + lane;
        if (k < K4) {
          wv[u] = ((const float4*)w)[k];
#pragma unroll
          for (int i = 0; i < 8; ++i) av[u][i] = ((const float4*)a[i])[k];
        } else {
          wv[u] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int i = 0; i < 8; ++i) av[u][i] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          acc[i] += (av[u][i].x * wv[u].x + av[u][i].y * wv[u].y) + (av[u][i].z * wv[u].z + av[u][i].w * wv[u].w);
    }
  } else {
    for (int k = lane; k < K; k += 64) {
      const float wk = w[k];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += a[i][k] * wk;
    }
  }
  // sum over the lanes: the first three exchanges halve the rows a lane carries (4 + 2 + 1 + 3 exchanges instead of 8 x 6);
  // lanes 8 j .. 8 j + 7 end with row j
#pragma unroll
  for (int half = 4; half >= 1; half >>= 1) {
    const bool hi = lane & (8 * half);
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const float keep = hi ? acc[i + half] : acc[i], give = hi ? acc[i] : acc[i + half];
      acc[i] = keep + __shfl_xor(give, 8 * half, 64);
    }
  }
  float v = acc[0];
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int m = m0 + (lane >> 3);
  if ((lane & 7) == 0 && m < M) C[(size_t)out(m) * N + n] = v;
}

// The same product with what stands around it in a launch-bound fp32 layer (K a multiple of 4, operands on 16 bytes):
//   NORM   : A is the residual stream; its rows are normalised on the way in - the wave that multiplies a row holds all of it, so
//            the sum of squares falls out of the same loads, the gain goes into the weight and the row factor into the result;
//   F_RESID: C += A W^T (fresh: C = A W^T), the residual stream itself; an element belongs to one wave;
//   F_SWIGLU: a wave takes the gate column n and the up column N + n and writes silu(gate) * up;
//   F_QKV  : rotary embedding (the pair's other column is the neighbouring wave's), q in place, k and v into their cache slots.
// Row i of A is row i * in_stride + in_off.  Against a norm, an add and a swiglu launch of their own a layer takes 5 launches instead
// of 9; a launch is 3.5 us on the host and 2.5 to 4 on the GPU whatever it does (d 128: the loop of draft, similarity, verify and
// commit 349 us with 92 launches, 234 with 58).  Larger fp32 models are bound by the products themselves.
enum { F_STORE = 0, F_RESID = 1, F_SWIGLU = 2, F_QKV = 3 };
struct SmallQkv { float *kc, *vc; const float* rope_tab; int T, d, dh, S_cap, rope_pos; size_t row_stride, head_stride; PosDesc pos; TreeDesc tree; };
struct NoQkv {};
template <bool NORM, int EPI, typename QKV>
__global__ __launch_bounds__(256) void k_gemm_small(const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ g, float* C, int M,
                                                    int N, int K, float eps, int in_stride, int in_off, int fresh, RowMap out, QKV qkv) {
  constexpr int NC = EPI == F_SWIGLU ? 2 : 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = blockIdx.x * 4 + wave, m0 = blockIdx.y * 8;
  if (n >= N) return;
  const int m = m0 + (lane >> 3);          // the row whose result this lane ends with
  const bool owner = (lane & 7) == 0 && m < M;
  float old = 0.f;
  if (EPI == F_RESID && owner && !fresh) old = C[(size_t)m * N + n];
  // F_QKV: N = 3 d is a multiple of 4, so all waves of a workgroup are here; position and rotary factor while the operands come
  int r = 0, sec = 0, slot = 0, img = -1;
  float2 f = make_float2(1.f, 0.f);
  if constexpr (EPI == F_QKV) {
    r = min(m, M - 1) / qkv.T;
    sec = n / qkv.d;
    token_pos(qkv.pos, qkv.tree, r, min(m, M - 1) - r * qkv.T, &slot, &img);
  }
  const float4 *w[NC], *a[8];
#pragma unroll
  for (int c = 0; c < NC; ++c) w[c] = (const float4*)(W + (size_t)(c * N + n) * K);
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = (const float4*)(A + ((size_t)min(m0 + i, M - 1) * in_stride + in_off) * K);
  float acc[NC + (NORM ? 1 : 0)][8];       // the columns' products, then the sums of squares
#pragma unroll
  for (auto& row : acc)
#pragma unroll
    for (int i = 0; i < 8; ++i) row[i] = 0.f;
  const int K4 = K >> 2;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k0 = 0; k0 < K4; k0 += 128) {
    float4 wv[2][NC], gv[2], av[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 1 && k0 + 64 >= K4) break;    // (uniform)
      const int k = min(k0 + 64 * u + lane, K4 - 1);   // lanes past the end repeat the last piece
#pragma unroll
      for (int c = 0; c < NC; ++c) wv[u][c] = w[c][k];
      if constexpr (NORM) gv[u] = ((const float4*)g)[k];
#pragma unroll
      for (int i = 0; i < 8; ++i) av[u][i] = a[i][k];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 1 && k0 + 64 >= K4) break;
      if (k0 + 64 * u + lane >= K4) {        // ... and add nothing, not even where that piece holds an infinity
#pragma unroll
        for (int c = 0; c < NC; ++c) wv[u][c] = zero;
        if constexpr (NORM) gv[u] = zero;
#pragma unroll
        for (int i = 0; i < 8; ++i) av[u][i] = zero;
      }
      if constexpr (NORM) {
#pragma unroll
        for (int c = 0; c < NC; ++c) wv[u][c] = make_float4(wv[u][c].x * gv[u].x, wv[u][c].y * gv[u].y, wv[u][c].z * gv[u].z, wv[u][c].w * gv[u].w);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float4 x = av[u][i];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c][i] += (x.x * wv[u][c].x + x.y * wv[u][c].y) + (x.z * wv[u][c].z + x.w * wv[u][c].w);
        if constexpr (NORM) acc[NC][i] += (x.x * x.x + x.y * x.y) + (x.z * x.z + x.w * x.w);
      }
    }
  }
  if constexpr (EPI == F_QKV) {
    if (img >= 0 && sec < 2) {
      const int half = qkv.dh >> 1, e = n % qkv.dh, pv = e >= half ? img % qkv.pos.grid_w : min(img / qkv.pos.grid_w, qkv.rope_pos - 1);
      f = *(const float2*)(qkv.rope_tab + ((size_t)pv * (qkv.dh >> 2) + ((e % half) >> 1)) * 2);
    }
  }
  // sums over the lanes; lanes 8 j .. 8 j + 7 end with row j.  The first three steps halve the rows a lane carries (a row swap exchanges
  // what two registers' halves do not keep), the last three add inside 8 lanes (as wave_reduce)
#pragma unroll
  for (auto& row : acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uintx2_t p = __builtin_amdgcn_permlane32_swap(__float_as_uint(row[i]), __float_as_uint(row[i + 4]), false, false);
      row[i] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uintx2_t p = __builtin_amdgcn_permlane16_swap(__float_as_uint(row[i]), __float_as_uint(row[i + 2]), false, false);
      row[i] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
    const bool hi = lane & 8;
    row[0] = (hi ? row[1] : row[0]) + dpp_move<0x128>(hi ? row[0] : row[1]);   // row_ror:8
    row[0] += dpp_move<0x141>(row[0]);     // row_half_mirror
    row[0] += dpp_move<0x4E>(row[0]);      // quad_perm:[2,3,0,1]
    row[0] += dpp_move<0xB1>(row[0]);      // quad_perm:[1,0,3,2]
  }
  if constexpr (EPI == F_QKV) {
    __shared__ float col[4][8];
    const float v = acc[0][0] / sqrtf(acc[NC][0] / (float)K + eps);
    if ((lane & 7) == 0) col[wave][lane >> 3] = v;
    __syncthreads();
    if (!owner) return;
    const float p = col[wave ^ 1][lane >> 3], w0 = n & 1 ? p * f.y + v * f.x : v * f.x - p * f.y;
    const int nd = n - sec * qkv.d, hd = nd / qkv.dh, e = nd % qkv.dh;
    const size_t head = (size_t)r * qkv.row_stride + (size_t)hd * qkv.head_stride;
    if (sec == 0) C[(size_t)m * qkv.d + nd] = w0;
    else if (slot >= 0 && slot < qkv.S_cap) {
      if (sec == 1) qkv.kc[head + k_index(slot, e, qkv.dh)] = w0;
      else qkv.vc[head + v_index(slot, e, qkv.dh)] = v;
    }
    return;
  }
  if (!owner) return;
  const float scale = NORM ? 1.0f / sqrtf(acc[NC][0] / (float)K + eps) : 1.f;
  const float v = acc[0][0] * scale;
  if constexpr (EPI == F_SWIGLU) C[(size_t)m * N + n] = v / (1.0f + expf(-v)) * (acc[NC - 1][0] * scale);
  else if constexpr (EPI == F_RESID) C[(size_t)m * N + n] = old + v;
  else C[(size_t)out(m) * N + n] = v;
}

template <bool NORM, int EPI, typename QKV = NoQkv>
static void gemm_small(Ctx* c, const float* A, const char* W, const char* g, float* C, int M, int N, int K, hipStream_t s, int fresh = 0,
                       RowMap out = RowMap{}, int in_stride = 1, int in_off = 0, const QKV& qkv = QKV{}) {
  Timed timed(c, VVS_K_GEMM, s);
  hipLaunchKernelGGL((k_gemm_small<NORM, EPI, QKV>), dim3((N + 3) / 4, (M + 7) / 8), dim3(256), 0, s, A, (const float*)W, (const float*)g, C, M, N, K,
                     c->cfg.rms_eps, in_stride, in_off, fresh, out, qkv);
}

// C[splits][M][N] (fp32 partial sums) = A[M][K] * W[N][K]^T (bf16: both operands in packed fragment order)
static int run_gemm(Ctx* c, const void* A, const void* W, float* C, int M, int N, int K, GemmPlan p, hipStream_t s, RowMap out = RowMap{}) {
  Timed timed(c, VVS_K_GEMM, s);
  if (c->cfg.dtype == VVS_BF16) {
    mfma_gemm((const bf16_t*)A, (const bf16_t*)W, C, M, N, K, p, s, out);
    return p.splits;
  }
  dim3 grid((N + 3) / 4, (M + 7) / 8);
  if (K % 4 == 0 && ((uintptr_t)A | (uintptr_t)W) % 16 == 0)
    hipLaunchKernelGGL(k_gemm_simple<true>, grid, dim3(256), 0, s, (const float*)A, (const float*)W, C, M, N, K, out);
  else
    hipLaunchKernelGGL(k_gemm_simple<false>, grid, dim3(256), 0, s, (const float*)A, (const float*)W, C, M, N, K, out);
  return 1;
}

// ------------------------------------------------------------------------------------------------ one forward over T tokens per row
// bf16, enough rows that no projection needs a grid-level K split: 5 kernels per layer.  The residual
// stream is kept three ways by whoever updates it (embedding kernel, O / down epilogues): fp32 x,
// bf16(x * g) in packed operand order (g = gain of the norm that reads it next), and per-row sums of
// squares; the projections that follow a norm take bf16(x * g) as operand and apply the RMSNorm row
// factor to their output tile.  The packed weights are the caller's bf16 values, unchanged.
static void forward_fused(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int Tq, const int32_t* d_tokens_bt, const void* pc,
                          const void* pu, int chunk_start, const int32_t* forced, int n_forced, int logits_mode, hipStream_t s,
                          bool from_din) {
  const int d = c->d, F = c->F, M = c->R * Tq, NS = n_slabs(d);
  float* x = (float*)(c->ws + c->w.x);
  bf16_t* xb = (bf16_t*)(c->ws + c->w.h);
  float* ss = (float*)(c->ws + c->w.ss);
  bf16_t* attn = (bf16_t*)(c->ws + c->w.attn);
  bf16_t* act = (bf16_t*)(c->ws + c->w.act);
  EmbedArgs ea{Tq, d, c->V, d_tokens_bt ? 0 : 1, d_tokens_bt, pc, pu, c->cfg.prefix_kind, c->cfg.n_classes, c->P, chunk_start,
               n_forced, forced};
  const float* g_first = (const float*)(c->pw + c->p.layer0 + c->p.g1);   // gain of the first layer's first norm
  const float* gf = (const float*)(c->pw + c->p.gf);
  // verify calls of up to 64 tokens per row at head size 64: projection + attention in one launch, fed by the row-padded operand layout
  const bool few = layers_in_one_launch(c, Tq);
  const int pad = few ? 0 : mfma_qkv_attention_rows(c, pos, Tq);
  const bool qa = pad > 0;
  const int pad_T = qa ? Tq : 0;
  const GemmPlan pq = plan_qkv(c, M), pr = plan_resid(c, M), pg = plan_gate_up(c, M), pl = plan_gemm(c, M, c->veff, d);
  // what each launch's idle CUs read ahead for the next one (nothing where no XCD owns a weight tile)
  auto weights = [&](const void* w, int N, int K, const GemmPlan& p) {
    if (p.row_owner) return WeightPrefetch{};
    // at most 2.5 MB for each XCD: beside the activations more would only push itself out of its 4 MB L2
    const int blocks = (p.bn / 32) * (K / 16), most = 8 * std::max(1, 2560 / blocks);
    return WeightPrefetch{(const uint4*)w, std::min(N / p.bn, most), blocks, 1, 0, (M + p.bm - 1) / p.bm};
  };
  auto layer = [&](int l) { return c->pw + c->p.layer0 + c->p.layer_stride * l; };
  auto pf_qkv = [&](int l) {
    if (qa) return WeightPrefetch{(const uint4*)(layer(l) + c->p.wqkv), c->H, 2 * (d / 16), 3, (d / 32) * (d / 16), c->B};
    return weights(layer(l) + c->p.wqkv, 3 * d, d, pq);
  };
  if (few && from_din) {      // the input map is part of the launch
  } else if (from_din) {      // drafter: x = [embedding ; feature] W_fc
    Timed timed(c, VVS_K_GEMM, s);
    mfma_gemm_resid(c, (const bf16_t*)(c->ws + c->w.din), (const bf16_t*)(c->pw + c->p.fc), x, xb, ss, g_first, M, 2 * d, s, pf_qkv(0), pad_T, pad, true);
  } else {
    Timed timed(c, VVS_K_ELEMENTWISE, s);
    hipLaunchKernelGGL(k_embed_packed, dim3(M), dim3(256), 0, s, x, xb, ss, NS, (const bf16_t*)(c->pw + c->p.embed),
                       (const bf16_t*)(c->pw + c->p.prefix_embed), g_first, ea, pad_T, pad);
  }
  if (few) {
    Timed timed(c, VVS_K_GEMM, s);
    launch_layers_few(c, tree, pos, Tq, from_din, s);
  }
  for (int l = 0; l < c->L && !few; ++l) {
    const char* lw = c->pw + c->p.layer0 + c->p.layer_stride * l;
    if (qa) {
      Timed timed(c, VVS_K_GEMM, s);
      mfma_qkv_attention(c, l, xb, (const bf16_t*)(lw + c->p.wqkv), ss, tree, pos, Tq, s, weights(lw + c->p.wo, d, d, pr));
    } else {
      { Timed timed(c, VVS_K_GEMM, s);
        mfma_gemm_qkv(c, l, xb, (const bf16_t*)(lw + c->p.wqkv), ss, tree, pos, Tq, pq, s);
      }
      { Timed timed(c, VVS_K_ATTENTION, s);
        mfma_attention(c, l, tree, pos, Tq, s, weights(lw + c->p.wo, d, d, pr));
      }
    }
    { Timed timed(c, VVS_K_GEMM, s);
      mfma_gemm_resid(c, attn, (const bf16_t*)(lw + c->p.wo), x, xb, ss, (const float*)(lw + c->p.g2), M, d, s,
                      weights(lw + c->p.wgu, 2 * F, d, pg));
    }
    { Timed timed(c, VVS_K_GEMM, s);
      mfma_gemm_swiglu(c, xb, (const bf16_t*)(lw + c->p.wgu), act, ss, M, F, d, pg, s, weights(lw + c->p.wd, d, F, pr));
    }
    { Timed timed(c, VVS_K_GEMM, s);
      // the next reader of x is the next layer's first norm, or the final norm
      const float* g_next = l + 1 < c->L ? (const float*)(lw + c->p.layer_stride + c->p.g1) : gf;
      const WeightPrefetch next = l + 1 < c->L ? pf_qkv(l + 1) : logits_mode == 1 ? weights(c->pw + c->p.wout, c->veff, d, pl) : WeightPrefetch{};
      mfma_gemm_resid(c, act, (const bf16_t*)(lw + c->p.wd), x, xb, ss, g_next, M, F, s, next, l + 1 < c->L ? pad_T : 0, pad);
    }
  }
  if (logits_mode == 0) return;
  float* logits = (float*)(c->ws + c->w.logits);
  const bf16_t* wout = (const bf16_t*)(c->pw + c->p.wout);
  if (logits_mode == 1) {
    Timed timed(c, VVS_K_GEMM, s);
    mfma_gemm_scaled(c, xb, wout, logits, ss, M, c->veff, d, pl, s, RowMap{Tq, tree.all, tree.first});
  } else {                    // last token of every row
    bf16_t* hf = (bf16_t*)(c->ws + c->w.hf);
    float* ss2 = (float*)(c->ws + c->w.ss2);
    { Timed timed(c, VVS_K_ELEMENTWISE, s);
      hipLaunchKernelGGL(k_gather_rows, dim3(c->R), dim3(256), 0, s, x, ss, gf, hf, ss2, d, NS, Tq, Tq - 1);
    }
    Timed timed(c, VVS_K_GEMM, s);
    mfma_gemm_scaled(c, hf, wout, logits, ss2, c->R, c->veff, d, plan_gemm(c, c->R, c->veff, d), s);
  }
}

// fp32, few rows of a narrow model: 5 launches per layer.
static void forward_small(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int Tq, const int32_t* d_tokens_bt, const void* pc, const void* pu,
                          int chunk_start, const int32_t* forced, int n_forced, int logits_mode, hipStream_t s, bool from_din) {
  const int d = c->d, F = c->F, M = c->R * Tq;
  float* x = (float*)(c->ws + c->w.x);
  float* q = (float*)(c->ws + c->w.q);
  float* attn = (float*)(c->ws + c->w.attn);
  float* act = (float*)(c->ws + c->w.act);
  if (from_din) {             // drafter: x = [embedding ; feature] W_fc
    gemm_small<false, F_RESID>(c, (const float*)(c->ws + c->w.din), c->pw + c->p.fc, nullptr, x, M, d, 2 * d, s, 1);
  } else {
    Timed timed(c, VVS_K_ELEMENTWISE, s);
    EmbedArgs ea{Tq, d, c->V, d_tokens_bt ? 0 : 1, d_tokens_bt, pc, pu, c->cfg.prefix_kind, c->cfg.n_classes, c->P, chunk_start, n_forced, forced};
    hipLaunchKernelGGL(k_embed<float>, dim3(M), dim3(256), 0, s, x, (const float*)(c->pw + c->p.embed), (const float*)(c->pw + c->p.prefix_embed), ea);
  }
  for (int l = 0; l < c->L; ++l) {
    const char* lw = c->pw + c->p.layer0 + c->p.layer_stride * l;
    float *kc = (float*)c->kv + c->kv_layer_stride * l, *vc = kc + c->kv_v_off;
    gemm_small<true, F_QKV>(c, x, lw + c->p.wqkv, lw + c->p.g1, q, M, 3 * d, d, s, 0, RowMap{}, 1, 0,
                            SmallQkv{kc, vc, (const float*)(c->ws + c->w.rope_tab), Tq, d, c->dh, c->S_cap, c->rope_pos, c->kv_row_stride,
                                     c->kv_head_stride, pos, tree});
    { Timed timed(c, VVS_K_ATTENTION, s);
      hipLaunchKernelGGL(k_attn_simple, dim3(Tq, c->H, c->R), dim3(256), sizeof(float) * (c->S_cap + 16), s, q, kc, vc, attn, tree, pos, Tq, d, c->dh,
                         c->kv_row_stride, c->kv_head_stride, c->S_cap);
    }
    gemm_small<false, F_RESID>(c, attn, lw + c->p.wo, nullptr, x, M, d, d, s);
    gemm_small<true, F_SWIGLU>(c, x, lw + c->p.wgu, lw + c->p.g2, act, M, F, d, s);
    gemm_small<false, F_RESID>(c, act, lw + c->p.wd, nullptr, x, M, d, F, s);
  }
  if (logits_mode == 0) return;
  float* logits = (float*)(c->ws + c->w.logits);
  const char *wout = c->pw + c->p.wout, *gf = c->pw + c->p.gf;
  if (logits_mode == 1) gemm_small<true, F_STORE>(c, x, wout, gf, logits, M, c->veff, d, s, 0, RowMap{Tq, tree.all, tree.first});
  else gemm_small<true, F_STORE>(c, x, wout, gf, logits, c->R, c->veff, d, s, 0, RowMap{}, Tq, Tq - 1);   // last token of every row
}

template <typename T>
static void forward_t(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int Tq, const int32_t* d_tokens_bt, const void* pc,
                      const void* pu, int chunk_start, const int32_t* forced, int n_forced, int logits_mode, hipStream_t s,
                      bool from_din) {
  const int d = c->d, F = c->F, M = c->R * Tq;
  if (plan_fused(c, M)) {
    forward_fused(c, tree, pos, Tq, d_tokens_bt, pc, pu, chunk_start, forced, n_forced, logits_mode, s, from_din);
    return;
  }
  // The limits are where the parity tests of the small layer end, not where it stops paying.  Step of 3 layers, plain / small, us: at the limits
  // d 1024, d_ff 4096, 128 rows 1014 / 824; beyond each, 256 rows (d 1024, d_ff 2752) 1405 / 1222, d 1280 (128 rows) 1205 / 1008, d_ff 5504
  // (128 rows) 1297 / 1029; well inside, d 128 with 10 rows 138 / 91.
  if (sizeof(T) == 4 && M <= 128 && d <= 1024 && F <= 4096) {
    forward_small(c, tree, pos, Tq, d_tokens_bt, pc, pu, chunk_start, forced, n_forced, logits_mode, s, from_din);
    return;
  }
  float* x = (float*)(c->ws + c->w.x);
  T* h = (T*)(c->ws + c->w.h);
  float* go = (float*)(c->ws + c->w.gemm_out);
  T* q = (T*)(c->ws + c->w.q);
  T* attn = (T*)(c->ws + c->w.attn);
  T* act = (T*)(c->ws + c->w.act);
  const float* rope = (const float*)(c->ws + c->w.rope_tab);
  EmbedArgs ea{Tq, d, c->V, d_tokens_bt ? 0 : 1, d_tokens_bt, pc, pu, c->cfg.prefix_kind, c->cfg.n_classes, c->P, chunk_start,
               n_forced, forced};
  int splits = 0;   // partial sums waiting to be added to x
  size_t sstride = 0;
  if (from_din) {             // drafter: x = 0 + [embedding ; feature] W_fc, added by the first norm kernel
    launch_fill_zero(x, sizeof(float) * (size_t)M * d, s);
    splits = run_gemm(c, c->ws + c->w.din, c->pw + c->p.fc, go, M, d, 2 * d, plan_partial(c, M, d, 2 * d), s);
    sstride = (size_t)M * d;
  } else {
    Timed timed(c, VVS_K_ELEMENTWISE, s);
    hipLaunchKernelGGL(k_embed<T>, dim3(M), dim3(256), 0, s, x, (const T*)(c->pw + c->p.embed),
                       (const T*)(c->pw + c->p.prefix_embed), ea);
  }
  const bool wide = layers_in_one_launch(c, Tq);
  if (wide) {
    Timed timed(c, VVS_K_GEMM, s);
    launch_layers_wide(c, tree, pos, Tq, s);
    splits = kFewWideShares;
    sstride = (size_t)M * d;
  }
  for (int l = 0; l < c->L && !wide; ++l) {
    const char* lw = c->pw + c->p.layer0 + c->p.layer_stride * l;
    T* kc = (T*)c->kv + c->kv_layer_stride * l;
    T* vc = (T*)c->kv + c->kv_v_off + c->kv_layer_stride * l;
    { Timed timed(c, VVS_K_ELEMENTWISE, s);
    launch_add_rmsnorm<T>(M, x, go, splits, sstride, d, (const float*)(lw + c->p.g1), c->cfg.rms_eps, h, 1, 0, s);
    }
    int sp;
    GemmPlan pq = plan_qkv(c, M);
    // with 160+ tiles an unsplit projection streams its weights as fast as a split one, and its epilogue
    // does the rotary embedding and the cache write: one kernel less
    if (pq.splits > 1 && ((M + pq.bm - 1) / pq.bm) * (3 * d / pq.bn) >= 160) pq.splits = 1;
    if (c->cfg.dtype == VVS_BF16 && pq.splits == 1) {
      Timed timed(c, VVS_K_GEMM, s);           // projection + rotary + cache write in one kernel
      mfma_gemm_qkv(c, l, (const bf16_t*)h, (const bf16_t*)(lw + c->p.wqkv), nullptr, tree, pos, Tq, pq, s);
    } else {
      sp = run_gemm(c, h, lw + c->p.wqkv, go, M, 3 * d, d, pq, s);
      Timed timed(c, VVS_K_ELEMENTWISE, s);
      hipLaunchKernelGGL(k_rope_kv<T>, dim3(M, ((d >> 1) + 255) / 256), dim3(256), 0, s, go, sp, (size_t)M * 3 * d, q, kc, vc, rope, tree, pos, Tq, d, c->dh,
                         c->kv_row_stride, c->kv_head_stride, c->S_cap, c->rope_pos);
    }
    if constexpr (sizeof(T) == 2) {
      Timed timed(c, VVS_K_ATTENTION, s);
      mfma_attention(c, l, tree, pos, Tq, s);
    } else {
      Timed timed(c, VVS_K_ATTENTION, s);
      size_t lds = sizeof(float) * (c->S_cap + 16);
      hipLaunchKernelGGL(k_attn_simple, dim3(Tq, c->H, c->R), dim3(256), lds, s, q, kc, vc, attn, tree, pos, Tq, d, c->dh,
                         c->kv_row_stride, c->kv_head_stride, c->S_cap);
    }
    sp = run_gemm(c, attn, lw + c->p.wo, go, M, d, d, plan_partial(c, M, d, d), s);
    { Timed timed(c, VVS_K_ELEMENTWISE, s);
    launch_add_rmsnorm<T>(M, x, go, sp, (size_t)M * d, d, (const float*)(lw + c->p.g2), c->cfg.rms_eps, h, 1, 0, s);
    }
    GemmPlan pg = plan_gate_up(c, M);
    if (c->cfg.dtype == VVS_BF16 && pg.splits == 1) {
      Timed timed(c, VVS_K_GEMM, s);           // projection + SwiGLU in one kernel
      mfma_gemm_swiglu(c, (const bf16_t*)h, (const bf16_t*)(lw + c->p.wgu), (bf16_t*)act, nullptr, M, F, d, pg, s, WeightPrefetch{});
    } else {
      sp = run_gemm(c, h, lw + c->p.wgu, go, M, 2 * F, d, pg, s);
      size_t n = (size_t)M * (F / 8);
      Timed timed(c, VVS_K_ELEMENTWISE, s);
      hipLaunchKernelGGL(k_swiglu<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, go, sp, (size_t)M * 2 * F, act, M, F,
                         c->cfg.dtype == VVS_BF16 ? 1 : 0);
    }
    splits = run_gemm(c, act, lw + c->p.wd, go, M, d, F, plan_partial(c, M, d, F), s);
    sstride = (size_t)M * d;
  }
  if (logits_mode == 0) return;
  T* hf = (T*)(c->ws + c->w.hf);
  float* logits = (float*)(c->ws + c->w.logits);
  const float* gf = (const float*)(c->pw + c->p.gf);
  int Ml;
  if (logits_mode == 1) {     // every token
    Ml = M;
    { Timed timed(c, VVS_K_ELEMENTWISE, s);
    launch_add_rmsnorm<T>(Ml, x, go, splits, sstride, d, gf, c->cfg.rms_eps, hf, 1, 0, s);
    }
  } else {                    // last token of every row
    Ml = c->R;
    { Timed timed(c, VVS_K_ELEMENTWISE, s);
    launch_add_rmsnorm<T>(Ml, x, go, splits, sstride, d, gf, c->cfg.rms_eps, hf, Tq, Tq - 1, s);
    }
  }
  GemmPlan pl = plan_gemm(c, Ml, c->veff, d);
  pl.splits = 1;
  run_gemm(c, hf, c->pw + c->p.wout, logits, Ml, c->veff, d, pl, s, logits_mode == 1 ? RowMap{Tq, tree.all, tree.first} : RowMap{});
}

void launch_forward(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int T, const int32_t* d_tokens_bt, const void* pc,
                    const void* pu, int chunk_start, const int32_t* forced, int n_forced, int logits_mode, hipStream_t s, bool from_din) {
  if (c->cfg.dtype == VVS_BF16)
    forward_t<bf16_t>(c, tree, pos, T - tree.first, d_tokens_bt, pc, pu, chunk_start, forced, n_forced, logits_mode, s, from_din);
  else forward_t<float>(c, tree, pos, T - tree.first, d_tokens_bt, pc, pu, chunk_start, forced, n_forced, logits_mode, s, from_din);
}

// ------------------------------------------------------------------------------------------------ token-level feature cache
// Section 4.3 / Algorithm 2 "UpdateCache".  The features of n tokens of the last forward (rows
// r * Tq + node of the residual stream x) are appended to the ring of row r: a feature is
// rmsnorm(x) * gf - the input of the output head - or x itself (pre_norm), stored like an activation
// of the model.  Ring state per row: (entries held, slot of the oldest); the token appended as the
// k-th since the oldest goes to slot (oldest + held + k) % slots.  One workgroup per (row, appended
// token); only the last `slots` tokens of a push are written (older ones would be overwritten by it).
//   path != nullptr: commit - the tokens are path[b][0 .. accept_len[b]] (skipped for finished prompts); a slice of the launch
//                    that moves the cache, of which it needs nothing (a launch of its own: 5 us behind it);
//   path == nullptr: prefill - the single token fixed_node into an emptied ring (state written here).
struct PushArgs {
  const float *x, *gf;
  void* ring;
  int32_t* ring_state;
  const int32_t *accept_len, *next_token, *path, *ring_was;  // ring_was: ring_state before the commit
  int Tq, fixed_node, R, d, slots, pre_norm;
  float eps;
};

// row r, appended token `at`
template <typename T>
__device__ __forceinline__ void push_feature(const PushArgs& a, int r, int at) {
  __shared__ float red[16];
  const int b = r >> 1;
  int n = 1, held = 0, oldest = 0;
  if (a.path) {
    if (a.next_token[b] < 0) return;
    n = a.accept_len[b] + 1;
    held = a.ring_was[r];
    oldest = a.ring_was[a.R + r];
  }
  const int i = max(0, n - a.slots) + at;
  if (i >= n) return;
  const int node = a.path ? a.path[b * VVS_MAX_T + i] : a.fixed_node;
  const float* xr = a.x + ((size_t)r * a.Tq + node) * a.d;
  float scale = 1.f;
  if (!a.pre_norm) {
    float ss = 0.f;
    for (int k = threadIdx.x; k < a.d; k += blockDim.x) ss += xr[k] * xr[k];
    ss = block_sum(ss, red);
    scale = 1.0f / sqrtf(ss / (float)a.d + a.eps);
  }
  T* dst = (T*)a.ring + ((size_t)r * a.slots + (oldest + held + i) % a.slots) * a.d;
  for (int k = threadIdx.x; k < a.d; k += blockDim.x) st(dst + k, a.pre_norm ? xr[k] : xr[k] * scale * a.gf[k]);
  if (!a.path && threadIdx.x == 0) {
    a.ring_state[r] = 1;
    a.ring_state[a.R + r] = 0;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_push_features(PushArgs a) { push_feature<T>(a, blockIdx.x, blockIdx.y); }

static PushArgs push_args(Ctx* c, const int32_t* path, int Tq, int fixed_node) {
  const int32_t* oc = (const int32_t*)(c->ws + c->w.outcome);
  return PushArgs{(const float*)(c->ws + c->w.x), (const float*)(c->pw + c->p.gf), c->ws + c->w.ring, (int32_t*)(c->ws + c->w.ring_state), oc, oc + c->B, path, oc + (kOutcomeSnap + 2) * c->B,
                  Tq, fixed_node, c->R, c->d, c->cfg.feature_slots, c->cfg.feature_pre_norm, c->cfg.rms_eps};
}

// ------------------------------------------------------------------------------------------------ KV commit
// Slot S + path[i] moves to slot S + i for the accepted positions i = 1..a.  path is strictly
// increasing with path[i] >= i, so a destination is never a source of a later position.  A thread
// owns either one chunk (CT: 16 bytes, or one element when the head size does not allow that) of a K
// row or one V element of a head for every accepted position; it reads the sources of up to 8
// positions before it writes them, which leaves one memory round trip per 8 positions.
// One workgroup of a prompt advances its state; everybody reads the lengths as the verify found them (`was`: [2][B], then the rings), so nothing
// has to be over before.  (A launch of its own behind this one: 2 to 5 us.)
struct CommitState { int32_t *state, *ring_state; const int32_t* was; int slots, B; };
__device__ __forceinline__ void commit_state(const CommitState& c, int b, int accepted, int token) {
  const int n = accepted + 1, B = c.B, R = 2 * B;
  c.state[b] = c.was[b] + n;               // cached length
  c.state[B + b] = c.was[B + b] + n;       // emitted image tokens
  c.state[2 * B + b] = token;              // pending token
  if (c.slots > 0)                         // the feature rings of both rows took n more entries
    for (int r = 2 * b; r < 2 * b + 2; ++r) {
      const int held = c.was[2 * B + r], oldest = c.was[2 * B + R + r], now = min(held + n, c.slots);
      c.ring_state[r] = now;
      c.ring_state[R + r] = (oldest + held + n - now) % c.slots;
    }
}

template <typename T, typename CT>
__global__ __launch_bounds__(256) void k_commit_kv(T* __restrict__ kcache, T* __restrict__ vcache, CommitState cs,
                                                   const int32_t* __restrict__ accept_len, const int32_t* __restrict__ next_token,
                                                   const int32_t* __restrict__ path, int H, int dh, size_t layer_stride,
                                                   size_t row_stride, size_t head_stride, int S_cap, int n_layers, PushArgs push) {
  constexpr int CH = sizeof(CT) / sizeof(T);   // elements per K chunk
  __shared__ int s_src[VVS_MAX_T];
  const int r = blockIdx.x, l = blockIdx.y, b = r >> 1;
  if (l == n_layers) {                         // the slice behind the layers: the feature ring
    if ((int)blockIdx.z < push.slots) push_feature<T>(push, r, blockIdx.z);
    return;
  }
  if (next_token[b] < 0) return;
  const int S = cs.was[b], a = accept_len[b];
  if (threadIdx.x == 0 && l == 0 && blockIdx.z == 0 && !(r & 1)) commit_state(cs, b, a, next_token[b]);
  if (threadIdx.x < VVS_MAX_T) s_src[threadIdx.x] = path[b * VVS_MAX_T + threadIdx.x];
  __syncthreads();
  T* kb = kcache + l * layer_stride + r * row_stride;
  T* vb = vcache + l * layer_stride + r * row_stride;
  const int n_k = H * dh / CH, n_v = H * dh;
  for (int item = blockIdx.z * blockDim.x + threadIdx.x; item < n_k + n_v; item += gridDim.z * blockDim.x) {   // one item per thread
    if (item < n_k) {
      const int col = item * CH, hd = col / dh, e = col % dh;
      T* kh = kb + hd * head_stride;
      for (int i0 = 1; i0 <= a; i0 += 8) {
        CT tmp[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int i = min(i0 + k, a);
          tmp[k] = *(const CT*)(kh + k_index(min(S + s_src[i], S_cap - 1), e, dh));
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int i = i0 + k;
          if (i <= a && s_src[i] != i && S + s_src[i] < S_cap) *(CT*)(kh + k_index(S + i, e, dh)) = tmp[k];
        }
      }
    } else {
      const int col = item - n_k, hd = col / dh, e = col % dh;
      T* vh = vb + hd * head_stride;
      for (int i0 = 1; i0 <= a; i0 += 8) {
        T tmp[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int i = min(i0 + k, a);
          tmp[k] = vh[v_index(min(S + s_src[i], S_cap - 1), e, dh)];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int i = i0 + k;
          if (i <= a && s_src[i] != i && S + s_src[i] < S_cap) vh[v_index(S + i, e, dh)] = tmp[k];
        }
      }
    }
  }
}

void launch_commit(Ctx* c, hipStream_t s) {
  Timed timed(c, VVS_K_COMMIT, s);
  const int32_t* oc = (const int32_t*)(c->ws + c->w.outcome);
  const int32_t* accept_len = oc;
  const int32_t* next_token = oc + c->B;
  const int32_t* path = oc + 2 * c->B;
  const bool vec = (c->dh * c->esz) % 16 == 0;
  const int items = c->H * c->dh / (vec ? 16 / (int)c->esz : 1) + c->H * c->dh;   // K chunks + V elements per (row, layer)
  const int slots = std::max(c->cfg.feature_slots, 0);
  const PushArgs push = push_args(c, path, c->last_T, -1);
  const CommitState cs{(int32_t*)(c->ws + c->w.state), (int32_t*)(c->ws + c->w.ring_state), oc + kOutcomeSnap * c->B, c->cfg.feature_slots, c->B};
  dim3 grid(c->R, c->L + (slots > 0), std::max((items + 255) / 256, slots));
  if (c->cfg.dtype == VVS_BF16 && vec)
    hipLaunchKernelGGL((k_commit_kv<bf16_t, uint4>), grid, dim3(256), 0, s, (bf16_t*)c->kv, (bf16_t*)c->kv + c->kv_v_off, cs, accept_len,
                       next_token, path, c->H, c->dh, c->kv_layer_stride, c->kv_row_stride, c->kv_head_stride, c->S_cap, c->L, push);
  else if (c->cfg.dtype == VVS_BF16)
    hipLaunchKernelGGL((k_commit_kv<bf16_t, bf16_t>), grid, dim3(256), 0, s, (bf16_t*)c->kv, (bf16_t*)c->kv + c->kv_v_off, cs, accept_len,
                       next_token, path, c->H, c->dh, c->kv_layer_stride, c->kv_row_stride, c->kv_head_stride, c->S_cap, c->L, push);
  else if (vec)
    hipLaunchKernelGGL((k_commit_kv<float, uint4>), grid, dim3(256), 0, s, (float*)c->kv, (float*)c->kv + c->kv_v_off, cs, accept_len,
                       next_token, path, c->H, c->dh, c->kv_layer_stride, c->kv_row_stride, c->kv_head_stride, c->S_cap, c->L, push);
  else
    hipLaunchKernelGGL((k_commit_kv<float, float>), grid, dim3(256), 0, s, (float*)c->kv, (float*)c->kv + c->kv_v_off, cs, accept_len,
                       next_token, path, c->H, c->dh, c->kv_layer_stride, c->kv_row_stride, c->kv_head_stride, c->S_cap, c->L, push);
}

void launch_push_prefill_feature(Ctx* c, int T_last_chunk, hipStream_t s) {
  if (c->cfg.feature_slots < 1) return;
  const PushArgs push = push_args(c, nullptr, T_last_chunk, T_last_chunk - 1);
  if (c->cfg.dtype == VVS_BF16) hipLaunchKernelGGL(k_push_features<bf16_t>, dim3(c->R), dim3(256), 0, s, push);
  else hipLaunchKernelGGL(k_push_features<float>, dim3(c->R), dim3(256), 0, s, push);
}

template <typename T>
__global__ void k_read_features(const T* __restrict__ ring, const int32_t* __restrict__ ring_state, float* __restrict__ out,
                                int32_t* __restrict__ count, int R, int d, int slots) {
  const int r = blockIdx.x, j = blockIdx.y;                // j-th oldest entry of row r
  const int held = ring_state[r], oldest = ring_state[R + r];
  if (j == 0 && threadIdx.x == 0 && (r & 1) == 0) count[r >> 1] = held;
  const T* src = ring + ((size_t)r * slots + (oldest + j) % slots) * d;
  float* dst = out + ((size_t)r * slots + j) * d;
  for (int k = threadIdx.x; k < d; k += blockDim.x) dst[k] = j < held ? ld(src + k) : 0.f;
}

void launch_read_features(Ctx* c, float* d_features, int32_t* d_count, hipStream_t s) {
  const int32_t* rstate = (const int32_t*)(c->ws + c->w.ring_state);
  dim3 grid(c->R, c->cfg.feature_slots);
  if (c->cfg.dtype == VVS_BF16)
    hipLaunchKernelGGL(k_read_features<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)(c->ws + c->w.ring), rstate, d_features, d_count, c->R,
                       c->d, c->cfg.feature_slots);
  else
    hipLaunchKernelGGL(k_read_features<float>, grid, dim3(256), 0, s, (const float*)(c->ws + c->w.ring), rstate, d_features, d_count, c->R,
                       c->d, c->cfg.feature_slots);
}

__global__ void k_read_state(const int32_t* __restrict__ state, int32_t* __restrict__ out, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = state[i];
}

void launch_read_state(Ctx* c, int32_t* d_state, hipStream_t s) {
  int n = 3 * c->B;
  hipLaunchKernelGGL(k_read_state, dim3((n + 255) / 256), dim3(256), 0, s, (const int32_t*)(c->ws + c->w.state), d_state, n);
}

void launch_set_state(Ctx* c, const int32_t* d_state, hipStream_t s) {
  int n = 3 * c->B;
  hipLaunchKernelGGL(k_read_state, dim3((n + 255) / 256), dim3(256), 0, s, d_state, (int32_t*)(c->ws + c->w.state), n);
}

// ------------------------------------------------------------------------------------------------ inspection
__global__ void k_debug_logits(const float* __restrict__ logits, const float* __restrict__ probs_ws, float* __restrict__ raw,
                               float* __restrict__ mixed, float* __restrict__ probs, int B, int T, int veff, float scale) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t per = (size_t)T * veff, n = (size_t)B * per;
  if (i >= n) return;
  const size_t b = i / per, rem = i % per;
  const float lc = logits[(2 * b) * per + rem], lu = logits[(2 * b + 1) * per + rem];
  if (raw) { raw[(2 * b) * per + rem] = lc; raw[(2 * b + 1) * per + rem] = lu; }
  if (mixed) mixed[i] = lu + scale * (lc - lu);
  if (probs) probs[i] = probs_ws[i];
}

void launch_debug_logits(Ctx* c, float* raw, float* mixed, float* probs, hipStream_t s) {
  size_t n = (size_t)c->B * c->last_T * c->veff;
  hipLaunchKernelGGL(k_debug_logits, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const float*)(c->ws + c->w.logits),
                     (const float*)(c->ws + c->w.probs), raw, mixed, probs, c->B, c->last_T, c->veff, c->cfg.cfg_scale);
}

template <typename T>
__global__ void k_debug_kv(const T* __restrict__ kh, const T* __restrict__ vh, float* __restrict__ dk, float* __restrict__ dv, int n_slots,
                           int H, int dh, size_t head_stride) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t d = (size_t)H * dh;
  if (i >= (size_t)n_slots * d) return;
  const int slot = (int)(i / d), col = (int)(i % d), hd = col / dh, e = col % dh;
  dk[i] = ld(kh + hd * head_stride + k_index(slot, e, dh));
  dv[i] = ld(vh + hd * head_stride + v_index(slot, e, dh));
}

void launch_debug_kv(Ctx* c, int layer, int row, int n_slots, float* dk, float* dv, hipStream_t s) {
  size_t n = (size_t)n_slots * c->d;
  if (!n) return;
  size_t off = c->kv_layer_stride * layer + c->kv_row_stride * row;
  unsigned blocks = (unsigned)((n + 255) / 256);
  if (c->cfg.dtype == VVS_BF16)
    hipLaunchKernelGGL(k_debug_kv<bf16_t>, dim3(blocks), dim3(256), 0, s, (const bf16_t*)c->kv + off,
                       (const bf16_t*)c->kv + c->kv_v_off + off, dk, dv, n_slots, c->H, c->dh, c->kv_head_stride);
  else
    hipLaunchKernelGGL(k_debug_kv<float>, dim3(blocks), dim3(256), 0, s, (const float*)c->kv + off,
                       (const float*)c->kv + c->kv_v_off + off, dk, dv, n_slots, c->H, c->dh, c->kv_head_stride);
}

__global__ void k_sum_splits(const float* __restrict__ part, int splits, size_t n, float* __restrict__ out) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float v = 0.f;
  for (int s = 0; s < splits; ++s) v += part[s * n + i];
  out[i] = v;
}

void launch_debug_gemm(Ctx* c, int m, int n, int k, const void* a, const void* w, void* scratch, float* out, hipStream_t s) {
  char* wt = (char*)scratch;
  char* at = wt + align_up((size_t)n * k * c->esz, 256);
  float* part = (float*)(at + align_up((size_t)align_up(m, 32) * k * c->esz, 256));
  if (c->cfg.dtype == VVS_BF16) {
    transpose_into<bf16_t>(w, wt, k, n, n, 0, s);
    const size_t total = (size_t)((m + 31) >> 5) * (k >> 4) * 64;
    hipLaunchKernelGGL(k_pack_a, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (const bf16_t*)a, (uint4*)at, m, k);
    a = at;
  } else {
    transpose_into<float>(w, wt, k, n, n, 0, s);
  }
  int sp = run_gemm(c, a, wt, part, m, n, k, plan_partial(c, m, n, k), s);
  size_t cnt = (size_t)m * n;
  hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, part, sp, cnt, out);
}

}  // namespace vvs
