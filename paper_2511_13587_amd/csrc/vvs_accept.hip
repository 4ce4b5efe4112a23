// Acceptance stage: CFG logit mix, softmax, strict / relaxed accept test with residual resampling,
// path walk (Section 2, "Speculative Decoding"; tree verification as in Section 3).
//
// Every node of the draft tree is evaluated speculatively and in parallel - one workgroup per
// (prompt, node) computes "which child of this node is accepted, or which token is drawn if none
// is" - and whichever workgroup of a prompt is done last follows the accepted children from the root.
// The uniforms are indexed by node, so this equals the sequential procedure.
#include "vvs_device.h"

#include <limits.h>

// Phase marks: a profiling build may define VVS_PHASE_MARK(i) to record a time stamp; normally nothing.
#ifndef VVS_PHASE_MARK
#define VVS_PHASE_MARK(i)
#endif

namespace vvs {

struct WalkOut {
  int32_t *accept_len, *path, *next_token, *keep;          // each may be nullptr; keep: the outcome for the commit
  const int32_t *state, *ring_state;                       // with keep: what the commit starts from
};

// Follows accepted children from the root: lane i of the wave holds the result of node i (accepted child or 0, token) and ends with path entry i.
__device__ __forceinline__ void walk_path(int child, int token, int b, int B, const WalkOut& o) {
  static_assert(VVS_MAX_T == 64, "one lane per node and path entry");
  const int i = threadIdx.x & 63;
  int cur = 0, a = 0, mine = 0;
  while (a < VVS_MAX_T - 1) {
    const int nxt = __builtin_amdgcn_readlane(child, cur);
    if (nxt <= cur) break;                 // 0 = nothing accepted (children always have larger ids)
    cur = nxt;
    if (i == ++a) mine = cur;
  }
  int tok = __builtin_amdgcn_readlane(token, cur);
  if (tok == kGaveUp) a = tok = -1;        // nothing is known of this prompt: no path, and no commit
  if (i == 0) {
    if (o.accept_len) o.accept_len[b] = a;
    if (o.next_token) o.next_token[b] = tok;
    if (o.keep) { o.keep[b] = a; o.keep[B + b] = tok; }
  }
  if (o.keep && i < 6) {                   // cached length, emitted tokens; held and oldest of both rows
    const int at = i < 2 ? i * B + b : (i >> 1) * 2 * B - 2 * B + 2 * b + (i & 1);
    o.keep[kOutcomeSnap * B + (i < 2 ? at : 2 * B + at)] = i < 2 ? o.state[at] : o.ring_state[at];
  }
  const int v = i <= a ? mine : -1;
  if (o.path) o.path[b * VVS_MAX_T + i] = v;
  if (o.keep) o.keep[2 * B + b * VVS_MAX_T + i] = v;
}

struct AcceptArgs {
  const float* logits;        // [R][T][veff]
  const int32_t* draft;       // [B][N]
  const float* q;             // [B][T][veff]
  const float* u;             // uniforms; element (b, j, which) at b*usb + j*usj + {uoa | uot}
  int usb, usj, uoa, uot;
  const int32_t* nbr;         // [vocab][relax_k] or nullptr
  const int32_t* n_emitted;   // [B] or nullptr (no cap, never finished)
  float* probs;               // [B][T][veff] out: target distributions
  float* work;                // [B][T][2][veff] scratch: running target P and draft Q
  int32_t* node_result;       // [B][VVS_MAX_T][2] out: (accepted child or 0, drawn token or -1)
  uint32_t* done;             // [B][kWalkLine] nodes of a prompt that are done, zero between calls; nullptr: the walk is a launch of its own
  const uint32_t* gave_up;    // not zero: the logits are not valid; or nullptr
  WalkOut out;
  int B;
  int T, veff, lo, mode, relax_k, G;
  float scale, delta;
};

// Largest 2 * veff * 4 bytes that is kept in LDS (160 KiB per CU, a few hundred bytes are static).
constexpr size_t kAcceptLdsMax = 144 * 1024;

// Inverse CDF in ascending id: first id whose running sum exceeds u * total; if rounding runs past
// the end, the last id with mass.  Each thread owns a contiguous chunk.
template <int CK>
__device__ int inverse_cdf(const float* __restrict__ P, int n, float u, float* red, int* ired, float* scan) {
  const int nt = blockDim.x, tid = threadIdx.x;
  const int per = (n + nt - 1) / nt;
  const int beg = min(tid * per, n), end = min(beg + per, n);
  // chunks of up to CK ids are read once into registers (16-byte reads when the chunk is aligned)
  float c[CK];
  const bool in_regs = per <= CK;
  float local = 0.f;
  if (in_regs) {
    if ((per & 3) == 0 && (n & 3) == 0) {
#pragma unroll
      for (int i = 0; i < CK; i += 4) {
        float4 v4 = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < per && beg + i < end) v4 = *(const float4*)(P + beg + i);
        c[i] = v4.x; c[i + 1] = v4.y; c[i + 2] = v4.z; c[i + 3] = v4.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < CK; ++i) c[i] = (beg + i < end) ? P[beg + i] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < CK; ++i) local += c[i];               // ids past the chunk hold 0
  } else {
    for (int v = beg; v < end; ++v) local += P[v];
  }
  // exclusive scan of the per-thread sums: inclusive inside a wave, then wave offsets in order
  float inc = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    float t = __shfl_up(inc, o, 64);
    if ((tid & 63) >= o) inc += t;
  }
  const int w = tid >> 6, nw = nt >> 6;
  __syncthreads();
  if ((tid & 63) == 63) scan[w] = inc;
  __syncthreads();
  float woff = 0.f, total = 0.f;
  for (int i = 0; i < nw; ++i) {
    if (i < w) woff += scan[i];
    total += scan[i];
  }
  const float target = u * total;
  float run = woff + inc - local;
  int cand = INT_MAX, last_pos = -1;
  if (in_regs) {
#pragma unroll
    for (int i = 0; i < CK; ++i) {
      const float pv = c[i];
      run += pv;
      if (beg + i < end) {
        if (pv > 0.f) last_pos = beg + i;
        if (cand == INT_MAX && run > target) cand = beg + i;
      }
    }
  } else {
    for (int v = beg; v < end; ++v) {
      const float pv = P[v];
      run += pv;
      if (pv > 0.f) last_pos = v;
      if (cand == INT_MAX && run > target) cand = v;
    }
  }
  int win = block_min_int(cand, ired);
  if (win == INT_MAX) win = block_max_int(last_pos, ired);
  (void)red;
  return win;
}

// LDS_PQ: the running target and draft distributions of the node live in (dynamic) LDS, 2 * veff
// floats; otherwise in the global scratch rows.
// A workgroup per CU and no second round: what counts is the chain of memory round trips inside a workgroup.  Both logit rows,
// the draft row of a node whose children are tested, and those children's ids and uniforms are all requested before the first
// is used.  WIDE (a slice of a multiple of 4 ids, rows on 16 bytes): a thread owns groups of 4 consecutive ids and moves 16 bytes
// at a time.  8 prompts x 27 nodes x 16384 ids: 26.6 us with 4-byte loads and the draft row asked for behind the softmax, 25.2 us so.
// Relaxed (the target goes through LDS once per tested child), 32 x 61 x 16384: 265 us and 243.
// The last node of a prompt walks: as a launch behind this one the walk took 4 to 5 us, so 3 (the whole call above 25.2 -> 24.0).
// NT threads, up to RK ids each (launch_accept_on chooses).
template <bool LDS_PQ, bool WIDE, int NT, int RK>
__global__ __launch_bounds__(NT, NT == 512 ? 4 : 1) void k_accept_node(AcceptArgs a, TreeDesc tree) {
  extern __shared__ __align__(16) float pq_lds[];
  __shared__ float red[32];
  __shared__ int ired[16];
  __shared__ float scan[16];
  __shared__ float nb_mass[64];
  __shared__ int nb_id[64];
  __shared__ float sh_num, sh_px, sh_qx;
  __shared__ int sh_m;
  __shared__ int sh_cx[VVS_MAX_T];         // drafted ids (inside the slice) and accept uniforms of this node's children, in order
  __shared__ float sh_cu[VVS_MAX_T];
  __shared__ int sh_cn[VVS_MAX_T], sh_nc;  // their node ids; how many
  __shared__ int sh_last;
  VVS_PHASE_MARK(0);
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  constexpr int nt = NT;
  const int T = a.T, V = a.veff;
  const float* lc = a.logits + ((size_t)(2 * b) * T + j) * V;
  const float* lu = a.logits + ((size_t)(2 * b + 1) * T + j) * V;
  float* P = LDS_PQ ? pq_lds : a.work + ((size_t)(b * T + j) * 2) * V;
  float* Q = P + V;
  float* prow = a.probs + (size_t)(b * T + j) * V;

  // CFG mix + softmax (temperature 1) over the allowed slice.  Up to RK ids per thread (the usual
  // codebook sizes): thread tid owns ids tid + k * nt and keeps its part of the running target (and
  // later of the draft distribution) in registers for the whole kernel; the LDS / global copy P is
  // only brought up to date where ids are addressed at random (relaxed neighbourhoods, the final
  // inverse-CDF draw).  Larger slices take the generic loops over P and Q.
  const bool regs = V <= RK * nt;
  auto id_of = [&](int k) { return WIDE ? ((k >> 2) * nt + tid) * 4 + (k & 3) : tid + k * nt; };
  auto load_row = [&](const float* row, float (&v)[RK]) {    // clamped: ids past the slice repeat the last ones
    if constexpr (WIDE) {
#pragma unroll
      for (int k = 0; k < RK; k += 4) {
        const float4 w = ((const float4*)row)[min((k >> 2) * nt + tid, (V >> 2) - 1)];
        v[k] = w.x; v[k + 1] = w.y; v[k + 2] = w.z; v[k + 3] = w.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < RK; ++k) v[k] = row[min(tid + k * nt, V - 1)];
    }
  };
  auto store_row = [&](float* row, const float (&v)[RK]) {
    if constexpr (WIDE) {
#pragma unroll
      for (int k = 0; k < RK; k += 4)
        if (id_of(k) < V) ((float4*)row)[(k >> 2) * nt + tid] = make_float4(v[k], v[k + 1], v[k + 2], v[k + 3]);
    } else {
#pragma unroll
      for (int k = 0; k < RK; ++k)
        if (id_of(k) < V) row[id_of(k)] = v[k];
    }
  };
  const bool tested = tree.first_child[j] > tree.n_forced;   // this node's children are tested (unless the image ends first)
  const int ne = a.n_emitted ? a.n_emitted[b] : 0;
  // the children (ascending node id = the order in which they are tried), their drafted ids and uniforms: one lane each
  const bool child = tested && tid < VVS_MAX_T && tid > 0 && tid < T && tree.parent[tid] == j;
  float p[RK], q[RK];
#pragma unroll
  for (int k = 0; k < RK; ++k) p[k] = q[k] = 0.f;
  float lcv[RK], luv[RK];
  if (regs) {
    load_row(lc, lcv);
    load_row(lu, luv);
    if (tested && RK == 16) load_row(a.q + (size_t)(b * T + j) * V, q);
  }
  // (a vector load behind the rows: a scalar one stood in front of them, 0.2 us of a call)
  const bool invalid = a.gave_up && __hip_atomic_load(a.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int child_x = 0;
  float child_u = 0.f;
  if (child) {
    child_x = min(max(a.draft[b * (T - 1) + tid - 1] - a.lo, 0), V - 1);
    child_u = a.u[(size_t)b * a.usb + (size_t)tid * a.usj + a.uoa];
  }
  if (regs) {
    float mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < RK; ++k) {
      p[k] = id_of(k) < V ? luv[k] + a.scale * (lcv[k] - luv[k]) : -INFINITY;
      mx = fmaxf(mx, p[k]);
    }
    if (tested && RK > 16) load_row(a.q + (size_t)(b * T + j) * V, q);   // (three rows at once do not fit the registers)
    mx = block_max(mx, red);
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < RK; ++k) {
      p[k] = id_of(k) < V ? expf(p[k] - mx) : 0.f;
      sum += p[k];
    }
    sum = block_sum(sum, red);
    const float inv_sum = 1.0f / sum;
#pragma unroll
    for (int k = 0; k < RK; ++k) {
      p[k] = p[k] * inv_sum;
      q[k] = id_of(k) < V ? q[k] : 0.f;
    }
    store_row(P, p);
    store_row(prow, p);
  } else {
    float mx = -INFINITY;
    for (int v = tid; v < V; v += nt) {
      const float m = lu[v] + a.scale * (lc[v] - lu[v]);
      P[v] = m;
      mx = fmaxf(mx, m);
    }
    mx = block_max(mx, red);
    float sum = 0.f;
    for (int v = tid; v < V; v += nt) {
      const float e = expf(P[v] - mx);
      P[v] = e;
      sum += e;
    }
    sum = block_sum(sum, red);
    for (int v = tid; v < V; v += nt) {
      const float pv = P[v] / sum;
      P[v] = pv;
      prow[v] = pv;
    }
  }
  if (tid < VVS_MAX_T) {                     // the first wave
    const unsigned long long m = __ballot(child);
    if (child) {
      const int rank = __popcll(m & ((1ull << tid) - 1ull));
      sh_cn[rank] = tid;
      sh_cx[rank] = child_x;
      sh_cu[rank] = child_u;
    }
    if (tid == 0) sh_nc = __popcll(m);
  }
  __syncthreads();

  VVS_PHASE_MARK(1);
  // this node's result; the last one of the prompt walks.  Results and counter with agent scope: the nodes run on all XCDs
  auto finish = [&](int child_id, int token) {
    int32_t* res = a.node_result + ((size_t)b * VVS_MAX_T + j) * 2;
    if (!a.done) {
      if (tid == 0) { res[0] = child_id; res[1] = token; }
      return;
    }
    uint32_t* done = a.done + (size_t)b * kWalkLine;
    if (tid == 0) {
      __hip_atomic_store((uint64_t*)res, (uint32_t)child_id | ((uint64_t)(uint32_t)token << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const bool last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)T - 1;
      if (last) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sh_last = last;
    }
    __syncthreads();
    if (!sh_last || tid >= VVS_MAX_T) return;
    uint64_t r = 0;
    if (tid < T) r = __hip_atomic_load((const uint64_t*)a.node_result + (size_t)b * VVS_MAX_T + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    walk_path((int)(uint32_t)r, (int)(uint32_t)(r >> 32), b, a.B, a.out);
  };
  int cap = INT_MAX;
  if (a.n_emitted) cap = a.G - ne - 1;
  if (cap < 0 || invalid) {                // image complete: nothing to accept, nothing to draw
    finish(0, cap < 0 ? -1 : kGaveUp);
    return;
  }

  int accepted = 0;
  bool p_in_memory = true;                   // P holds the current target (false: only the registers do)
  if (tree.first_child[j] >= 0 && tree.depth[j] < cap && tree.first_child[j] <= tree.n_forced) {
    accepted = tree.first_child[j];          // post verification: accepted without a test, nothing is read or changed
  } else if (tree.first_child[j] >= 0 && tree.depth[j] < cap) {
    const float* qrow = a.q + (size_t)(b * T + j) * V;
    if (!regs) {
      for (int v0 = tid; v0 < V; v0 += 8 * nt) {             // 8 independent requests per thread and pass
        float qv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) qv[k] = qrow[min(v0 + k * nt, V - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (v0 + k * nt < V) Q[v0 + k * nt] = qv[k];
      }
      __syncthreads();
    }
    const int n_children = sh_nc;
    for (int ci = 0; ci < n_children; ++ci) {
      const int c = sh_cn[ci];
      const int x = sh_cx[ci];
      const float ua = sh_cu[ci];
      const int xo = WIDE ? (x >> 2) % nt : x % nt, xk = WIDE ? (x >> 2) / nt * 4 + (x & 3) : x / nt;   // owner thread and register of id x
      if (a.mode == VVS_RELAXED && a.relax_k > 0) {
        // absorb neighbour mass in ascending distance while the absorbed total stays <= delta
        if (regs && !p_in_memory) {
          store_row(P, p);
          __syncthreads();
          p_in_memory = true;
        }
        if (tid < 64) {
          float pm = 0.f;
          int id = -1;
          if (tid < a.relax_k) {
            id = a.nbr[(size_t)(a.lo + x) * a.relax_k + tid] - a.lo;
            if (id >= 0 && id < V) pm = P[id]; else id = -1;
          }
          nb_mass[tid] = pm;
          nb_id[tid] = id;
        }
        __syncthreads();
        if (tid == 0) {
          float absorbed = 0.f;
          int m = 0;
          for (; m < a.relax_k; ++m) {
            if (nb_id[m] < 0) continue;
            if (absorbed + nb_mass[m] > a.delta) break;
            absorbed += nb_mass[m];
          }
          sh_m = m;
          sh_num = P[x] + absorbed;
        }
        __syncthreads();
        if (tid < sh_m && nb_id[tid] >= 0) P[nb_id[tid]] = 0.f;
        __syncthreads();
        if (tid == 0) P[x] = sh_num;
        __syncthreads();
        if (regs) {
#pragma unroll
          for (int k = 0; k < RK; ++k)
            if (id_of(k) < V) p[k] = P[id_of(k)];
        }
      }
      float num, qx;
      if (regs) {                                            // the owner of id x publishes its target and draft mass
        if (tid == xo) {
          float pv = 0.f, qv = 0.f;
#pragma unroll
          for (int k = 0; k < RK; ++k)
            if (k == xk) { pv = p[k]; qv = q[k]; }
          sh_px = pv;
          sh_qx = qv;
        }
        __syncthreads();
        num = sh_px;
        qx = sh_qx;
      } else {
        num = P[x];
        qx = Q[x];
      }
      if (ua * qx < num) { accepted = c; break; }
      // rejected: target <- normalised positive part of (target - draft); drop x from the draft
      if (regs) {
        float z = 0.f, zq = 0.f;
#pragma unroll
        for (int k = 0; k < RK; ++k) {
          z += fmaxf(0.f, p[k] - q[k]);
          zq += tid == xo && k == xk ? 0.f : q[k];
        }
        const float2 zz = block_sum2(z, zq, red);
        if (zz.x > 0.f) {                                    // a residual without mass leaves the target as it is
          const float inv = 1.0f / zz.x;                       // one division per row instead of one per id: 16 waves share 4 SIMDs
#pragma unroll
          for (int k = 0; k < RK; ++k) p[k] = fmaxf(0.f, p[k] - q[k]) * inv;
          p_in_memory = false;
        }
#pragma unroll
        for (int k = 0; k < RK; ++k)
          if (tid == xo && k == xk) q[k] = 0.f;                // x leaves the draft distribution
        if (!(zz.y > 0.f)) break;
        const float invq = 1.0f / zz.y;
#pragma unroll
        for (int k = 0; k < RK; ++k) q[k] = q[k] * invq;
      } else {
        float z = 0.f;
        for (int v = tid; v < V; v += nt) z += fmaxf(0.f, P[v] - Q[v]);
        z = block_sum(z, red);
        if (z > 0.f)
          for (int v = tid; v < V; v += nt) P[v] = fmaxf(0.f, P[v] - Q[v]) / z;
        __syncthreads();
        if (tid == 0) Q[x] = 0.f;
        __syncthreads();
        float zq = 0.f;
        for (int v = tid; v < V; v += nt) zq += Q[v];
        zq = block_sum(zq, red);
        if (!(zq > 0.f)) break;
        for (int v = tid; v < V; v += nt) Q[v] = Q[v] / zq;
        __syncthreads();
      }
    }
  }
  VVS_PHASE_MARK(2);
  if (accepted) {
    finish(accepted, -1);
    return;
  }
  if (regs && !p_in_memory) {                                // the draw addresses ids in ascending order: bring P up to date
    __syncthreads();
    store_row(P, p);
  }
  __syncthreads();
  const float ut = a.u[(size_t)b * a.usb + (size_t)j * a.usj + a.uot];
  const int tok = inverse_cdf<RK>(P, V, ut, red, ired, scan);
  VVS_PHASE_MARK(3);
  finish(0, a.lo + tok);
}

// The walk as a launch of its own: one wave per prompt.
__global__ __launch_bounds__(64) void k_walk(const int32_t* __restrict__ node_result, int B, int T, WalkOut out) {
  const int b = blockIdx.x, i = min((int)threadIdx.x, T - 1);
  const int2 r = ((const int2*)node_result)[(size_t)b * VVS_MAX_T + i];
  walk_path(r.x, r.y, b, B, out);
}

static void launch_accept_on(Ctx* c, const TreeDesc& tree, int T, const float* d_logits, const int32_t* d_draft_tokens, const float* d_q,
                             const float* d_u, int usb, int usj, int uoa, int uot, int mode, bool use_state, int32_t* d_accept_len,
                             int32_t* d_path, int32_t* d_next, int32_t* keep, const uint32_t* gave_up, float* probs, float* work, int32_t* node_result, uint32_t* done, hipStream_t s) {
  Timed timed(c, VVS_K_ACCEPT, s);
  AcceptArgs a;
  a.logits = d_logits; a.draft = d_draft_tokens; a.q = d_q; a.u = d_u;
  a.usb = usb; a.usj = usj; a.uoa = uoa; a.uot = uot;
  a.nbr = c->nbr;
  a.n_emitted = use_state ? (const int32_t*)(c->ws + c->w.state) + c->B : nullptr;
  a.probs = probs;
  a.work = work;
  a.node_result = node_result;
  a.done = done;
  a.gave_up = gave_up;
  a.out = WalkOut{d_accept_len, d_path, d_next, keep, (const int32_t*)(c->ws + c->w.state), (const int32_t*)(c->ws + c->w.ring_state)};
  a.B = c->B;
  a.T = T; a.veff = c->veff; a.lo = c->lo; a.mode = mode; a.relax_k = c->cfg.relax_k; a.G = c->G;
  a.scale = c->cfg.cfg_scale; a.delta = c->cfg.relax_delta;
  const size_t pq_bytes = (size_t)2 * c->veff * sizeof(float);
  // rows of a multiple of 4 ids that all start on 16 bytes
  const bool wide = c->veff % 4 == 0 && ((uintptr_t)a.logits | (uintptr_t)a.q | (uintptr_t)a.probs) % 16 == 0;
  const dim3 grid(T, c->B);
#define VVS_ACCEPT(LDS, NT, RK, BYTES)                                                                            \
  {                                                                                                               \
    const auto kernel = wide ? k_accept_node<LDS, true, NT, RK> : k_accept_node<LDS, false, NT, RK>;                \
    if ((BYTES) > 64 * 1024) allow_dynamic_lds((const void*)kernel, kAcceptLdsMax);                               \
    hipLaunchKernelGGL(kernel, grid, dim3(NT), (BYTES), s, a, tree);                                              \
  }
  // Few ids: 4 waves, which meet at a barrier sooner (1024 ids, one prompt of 5 nodes: 12.7 -> 8.4 us with the walk).  Many nodes: two workgroups of 512
  // threads to a CU cover each other's barriers, though 45 registers spill; the more a node does, the sooner.  Acceptance of 16384 ids, us, one of 1024 / two of 512:
  //   strict   8 x 41 nodes 36.6 / 37.2, 8 x 61 40.9 / 45.7, 12 x 61 57.3 / 59.6, 16 x 61 67.2 / 70.0, 17 x 61 72.0 / 75.4, 20 x 61 80.4 / 81.6, 32 x 41 90.0 / 88.5, 32 x 61 128.1 / 120.9
  //   relaxed  8 x 41 76.7 / 79.0, 8 x 61 99.4 / 102.1, 9 x 61 100.1 / 102.5, 10 x 61 116.8 / 109.7, 12 x 61 121.1 / 114.5, 16 x 61 132.9 / 128.8, 17 x 61 128.4 / 126.2, 20 x 61
  //     171 / 153, 32 x 61 224 / 189 (12 x 41, below the line, 88.4 / 83.7)
  const int many = mode == VVS_RELAXED && a.relax_k > 0 ? 576 : 1280;
  if (c->veff <= 4096) VVS_ACCEPT(true, 256, 16, pq_bytes / 2)
  else if (c->veff <= 16 * 1024 && T * c->B > many) VVS_ACCEPT(true, 512, 32, pq_bytes / 2)
  else if (c->veff <= 16 * 1024) VVS_ACCEPT(true, 1024, 16, pq_bytes / 2)
  else if (pq_bytes <= kAcceptLdsMax) VVS_ACCEPT(true, 1024, 16, pq_bytes)
  else {                                     // wider slices than the registers hold: the loops over ids
    hipLaunchKernelGGL((k_accept_node<false, false, 1024, 16>), grid, dim3(1024), 0, s, a, tree);
  }
#undef VVS_ACCEPT
  if (!done) hipLaunchKernelGGL(k_walk, dim3(c->B), dim3(64), 0, s, (const int32_t*)a.node_result, c->B, T, a.out);
}

void launch_accept(Ctx* c, const TreeDesc& tree, int T, const float* d_logits, const int32_t* d_draft_tokens, const float* d_q,
                   const float* d_u, int usb, int usj, int uoa, int uot, int mode, bool use_state, int32_t* d_accept_len,
                   int32_t* d_path, int32_t* d_next, bool keep_outcome, const uint32_t* gave_up, hipStream_t s) {
  launch_accept_on(c, tree, T, d_logits, d_draft_tokens, d_q, d_u, usb, usj, uoa, uot, mode, use_state, d_accept_len, d_path, d_next,
                   keep_outcome ? (int32_t*)(c->ws + c->w.outcome) : nullptr, gave_up, (float*)(c->ws + c->w.probs), (float*)(c->ws + c->w.pq_work),
                   (int32_t*)(c->ws + c->w.node_result), (uint32_t*)(c->ws + c->w.walk_sync), s);
}

// ------------------------------------------------------------------------------------------------ acceptance stage without any allocation
// The acceptance stage for callers that cannot allocate device memory and have no workspace to hand over: its
// two scratch buffers - the per-node results between k_accept_node and k_walk, and the per-node target
// distributions k_accept_node writes - live in one static device array.  Every GPU holds its own copy of the
// array at its own address; the address is looked up once per device (hipGetSymbolAddress, with that device
// current) and kept.  Nothing in the array has to start at zero: k_accept_node writes every entry that k_walk
// or a later phase reads.  Two calls that overlap on one GPU (two streams, two contexts) share the array and race.
constexpr size_t kNoAllocNodeBytes = (size_t)VVS_NOALLOC_MAX_PROMPTS * VVS_MAX_T * 2 * sizeof(int32_t);
constexpr size_t kNoAllocProbBytes = (size_t)VVS_NOALLOC_MAX_PROB_FLOATS * sizeof(float);
static __device__ __align__(256) unsigned char scratch[kNoAllocNodeBytes + kNoAllocProbBytes];

constexpr int kMaxDevices = 64;
static unsigned char* g_scratch_ptr[kMaxDevices];   // per device: address of that device's copy of `scratch`

vvs_status launch_accept_noalloc(Ctx* c, const TreeDesc& tree, int T, const float* d_logits, const int32_t* d_draft_tokens,
                                 const float* d_q, const float* d_u, int mode, int32_t* d_accept_len, int32_t* d_path, int32_t* d_next,
                                 hipStream_t s, std::string* err) {
  if (c->B > VVS_NOALLOC_MAX_PROMPTS || (size_t)c->B * T * c->veff > (size_t)VVS_NOALLOC_MAX_PROB_FLOATS) {
    *err = "accept_from_logits_noalloc: n_prompts * (n_nodes + 1) * V_eff exceeds VVS_NOALLOC_MAX_PROB_FLOATS (or n_prompts exceeds "
           "VVS_NOALLOC_MAX_PROMPTS): the static scratch array is too small for this call";
    return VVS_ESIZE;
  }
  if ((size_t)2 * c->veff * sizeof(float) > kAcceptLdsMax) {
    *err = "accept_from_logits_noalloc: the allowed-id slice is too wide for the LDS-resident acceptance kernel";
    return VVS_ESIZE;
  }
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) { *err = "accept_from_logits_noalloc: hipGetDevice failed"; return VVS_EHIP; }
  if (!g_scratch_ptr[dev]) {
    unsigned char* p = nullptr;
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      *err = std::string("accept_from_logits_noalloc: hipGetSymbolAddress: ") + hipGetErrorString(e);
      return VVS_EHIP;
    }
    g_scratch_ptr[dev] = p;
  }
  unsigned char* base = g_scratch_ptr[dev];
  launch_accept_on(c, tree, T, d_logits, d_draft_tokens, d_q, d_u, 2 * T, 2, 0, 1, mode, false, d_accept_len, d_path, d_next, nullptr, nullptr,
                   (float*)(base + kNoAllocNodeBytes), nullptr, (int32_t*)base, nullptr, s);
  return VVS_OK;
}

__global__ void k_prefill_finish(const int32_t* __restrict__ node_result, int32_t* __restrict__ state, int32_t* __restrict__ first,
                                 int B, int kv_len, int n_emitted, int grid) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int tok = node_result[((size_t)b * VVS_MAX_T) * 2 + 1];
  if (tok == kGaveUp) {                    // no image to continue: it counts as complete
    tok = -1;
    n_emitted = grid;
  }
  first[b] = tok;
  state[b] = kv_len;
  state[B + b] = n_emitted;
  state[2 * B + b] = tok;
}

void launch_prefill_finish(Ctx* c, int n_forced, int32_t* d_first, hipStream_t s) {
  hipLaunchKernelGGL(k_prefill_finish, dim3((c->B + 63) / 64), dim3(64), 0, s, (const int32_t*)(c->ws + c->w.node_result),
                     (int32_t*)(c->ws + c->w.state), d_first, c->B, c->P + n_forced, n_forced + 1, c->G);
}

}  // namespace vvs
