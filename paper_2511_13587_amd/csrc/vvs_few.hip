// bf16, few rows: all layers of a forward in ONE launch.
//
// A projection of few rows takes a few us whatever it computes: the launch, the first requests to HBM, the way down - and the next one
// starts cold behind it.  Here 256 workgroups (one per CU) stay for the whole forward and take its tiles in order; a tile's weights
// depend on nothing that the forward computes, so a workgroup asks for them at once and only then waits until the tiles of the phase
// before are done.
//
// Phases of a layer, each a list of tiles (one workgroup of 8 waves takes one; wide layers: k_layers_wide):
//   input map (drafter, once)   32 x 32 tiles of x = [embedding ; feature] W_fc
//   q/k/v                       32 x 32 tiles, rotary embedding, K / V cache write
//   attention                   16 or 32 queries of a head, 1, 2 or 4 rows
//   O                           32 x 32 tiles, x += tile
//   gate/up                     32 rows x 48 hidden units
//   down                        32 x 32 tiles, x += tile
// The waves of a tile split the contraction; their partial sums meet in LDS in a fixed order.
//
// How a phase hands on its results.  Every value that another workgroup reads is stored with agent scope (written through to the memory
// behind the L2s of the 8 XCDs); when a wave's stores are acknowledged and the workgroup has met at a barrier, one atomic counts the tile as done.
// A reader polls the counters with agent-scope loads.  Operands are then read by ordinary loads, through L1 and L2: every
// phase of every layer has buffers of its own (FewBuf), so that no cache can hold an older copy of an address - the launch itself began
// with clean caches.  The residual stream x is updated in place, each element by the owner of its tile, with agent-scope
// loads.  K and V of the call's own tokens are read by nobody before their counters say that they stand.
//   us per step, one launch per projection and for attention / one launch for all layers:  d 1280, 36 layers: 1 prompt x 27 tokens 1437 / 1046, 1 x 6
//   1311 / 950, 1 x 1 1304 / 944, 2 x 27 (108 rows) 1797 / 1490, 8 x 6 (96) 1807 / 1331, 3 x 27 (162) 1886 / 1743, 16 x 6 (192) 2157 / 2024; beyond: 4 x
//   27 (216 rows) 2027 / 2012, 2 x 61 (244) 2402 / 2274.  d 768, 12 layers: 4 x 6 396 / 311, 1 x 27 419 / 315, 3 x 27 (162) 448 / 415, 16 x 6 (192) 447 /
//   443.  Prefix and first tokens of the d 768 shape: 1 prompt x 1 token 336 / 267, 4 x 16 373 / 293, 32 x 1 404 / 300, 1 x 64 387 / 295.  Drafting calls of one layer, 5 pairs: 8 prompts, 26 nodes 460 / 402; 32 prompts (64 to 192 rows a level but the first) 634 / 623.  Where it
//   ends stands at few_rows.  (Tiles of two row-blocks, as wide layers have, do not carry it further: XL, 300 rows +8 %, 432 +25 %.)
//   A phase of 54 rows takes 4.3 to 7.2 us (8.5 before): 1.2 to 1.7 from the last tile counted to the next phase's first load, 1.5 to 3 for the operand
//   and the products, 1 for sum and epilogue, 0.5 to 0.8 until the stores are acknowledged.
//   Handing on alone, with 80 / 240 tiles of a phase: 1.3 / 2.4 us from one phase's last store to the next phase's first load; one
//   counter instead of eight 1.9 / 4.6, a flag per tile 2.9 / 4.8, release and acquire fences (an L2 write-back and invalidation) 27 / 32.
//
// Why no wait can last for ever.  The tiles are numbered in the order of the phases, a tile waits for tiles of lower numbers only, and
// a workgroup takes its tiles in ascending order: the lowest unfinished tile is always being worked on, if only the workgroup that
// owns it runs.  Where all workgroups of the launch are seen to run (they count themselves in at the start) tile t belongs to workgroup
// t % 256.  Where they do not within a bounded time - another program or stream keeps CUs, perhaps with a launch of this very
// kind that waits for the same CUs - nobody owns a tile beforehand: workgroups draw tile numbers from a counter, so that whoever runs
// works on the lowest one that is left.  Either way a wait also ends after FewArgs.polls looks: by then something else is broken, and what the
// forward leaves is not valid.  Its workgroups leave, the last one notes it (FewArgs.gave_up), and the kernels behind turn that into an outcome of
// its own: k_accept_node, k_prefill_finish, k_draft_select.
#include "vvs_mfma.h"

#include <algorithm>

namespace vvs {

enum { PH_INPUT = 0, PH_QKV, PH_ATTN, PH_O, PH_GU, PH_DOWN, PH_PART };
constexpr int kGroups = kFewGroups;
constexpr int kWaves = 8, kThreads = kWaves * 64;
// 100 MHz ticks that a workgroup waits for all others to be there.  They are within 3 us where nothing keeps a CU.  Drawn tiles cost 0 to 4 us a launch more
// than dealt ones (1 x 27 of the XL shape even 25 less), so waiting longer than that does not pay.  Prefix of one token, d 768, us, idle 278; while a kernel of
// another stream keeps 1 / 32 / 200 CUs: waiting 200 us 478 / 494 / 1038, 10 us 288 / 306 / 901, 5 us 282 / 299 / 670 (a launch each for projections and
// attention: idle 342, beside 1 CU 632).
constexpr long kAdmission = 500;

// ---- agent scope: written through, read from behind the L2s
__device__ __forceinline__ void put(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put(bf16_t* p, bf16_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put32(void* p, uint32_t v) { __hip_atomic_store((uint32_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put64(void* p, uint32_t lo, uint32_t hi) {
  __hip_atomic_store((uint64_t*)p, (uint64_t)lo | ((uint64_t)hi << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 get2(const float* p) {
  const uint64_t v = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}
__device__ __forceinline__ uint32_t get32(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void barrier() {          // of the workgroup; nothing moves across it
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

constexpr int kLine = kFewLine;
constexpr int kWideShares = kFewWideShares;

struct FewArgs {
  const char* layer0;                      // packed weights
  size_t layer_stride, o_g1, o_wqkv, o_wo, o_g2, o_wgu, o_wd;
  const float* gf;
  const bf16_t *fc, *din;                  // drafter: input map and its operand (else null)
  float* x;
  bf16_t* xb;                              // operand of the first layer and, afterwards, of the output head; ss: its sums of squares
  float* ss;
  char* buf;                               // FewBuf of every layer
  size_t buf_stride;
  bf16_t *kc, *vc;
  size_t kv_layer, kv_row, kv_head;
  const float* rope;
  uint32_t* sync;                          // kLine apart: how tiles are dealt (1: tile t to workgroup t % 256, 2: drawn), next tile to draw, eighths of the workgroups that
                                           // are done (beside it: workgroups that gave up a wait), [8] workgroups that are there, [8] done; then the layers' counters, then 8 of the input map
  uint32_t* gave_up;                       // not zero: a wait of this launch (drafter: or of an earlier level's) was given up
  int L, M, MT, T, d, H, F, R, NS, S_cap, rope_pos;
  int polls;                               // looks at a counter before a wait gives up
  int rows_per_unit;                       // rows that share an attention unit: 1, 2 or 4
  float* part;                             // wide layers: partial sums of O and of down [kWideShares][M][d]
  // SwiGLU by expf and a division, as k_swiglu has it: where gate/up as a launch of its own is split, whose sums that kernel takes.  Else by the
  // instructions for 2^x and 1 / x, as in the epilogue of whole sums (below a gate of -87.3 the latter's result is flushed to zero); d_ff 11008: 5 to 10 us
  // of 3000 less, 32 layers
  bool exact_gate;
  float eps, c_exp;
  PosDesc pos;
  TreeDesc tree;
};

// What a layer hands from phase to phase, rows padded to whole row-blocks
struct FewBuf {
  bf16_t *q, *att, *xb2, *act, *xb1;       // xb2: operand of gate/up, xb1: of the next layer's q/k/v
  float *ss2, *ss1;
};
__device__ __forceinline__ FewBuf few_buf(const FewArgs& a, int l) {
  char* p = a.buf + a.buf_stride * l;
  const size_t n = (size_t)a.MT * 32 * a.d;
  FewBuf b;
  b.q = (bf16_t*)p;
  b.att = b.q + n;
  b.xb2 = b.att + n;
  b.xb1 = b.xb2 + n;
  b.act = b.xb1 + n;
  b.ss2 = (float*)(b.act + (size_t)a.MT * 32 * a.F);
  b.ss1 = b.ss2 + (size_t)a.MT * 32 * a.NS;
  return b;
}

struct FewShared {
  int ticket, mode, stop, last;
};

// threadIdx.x, anew for every tile: what is computed from it would otherwise be kept in registers across all phases, and those are needed
__device__ __forceinline__ int few_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// The kernel's arguments, read anew for every tile: kept across all phases they would not fit the scalar registers
__device__ __forceinline__ const FewArgs& few_args() {
  typedef const FewArgs __attribute__((address_space(4)))* ptr;
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const FewArgs*)(ptr)p;
}

// Waits until lane i < n of wave 0 finds counter[i] at its own `want` (not zero); false: given up.
//   Pollers stand in the way of those who count: until one tile of the phase is done only one counter is looked at, about once per us.  36 layers of
//   54 rows, sleep 8 / 24 / 40 / 100 between two looks: 1028 / 1003 / 976 / 1030 us; counters 64 / 128 / 256 bytes apart 1052 / 1002 / 1003; a
//   sleep between the polls of all counters, or none for counters that are complete: no change.
__device__ __forceinline__ bool few_wait(const uint32_t* counter, int n, uint32_t want, FewShared* sh) {
  const int lane = threadIdx.x & 63;
  if (threadIdx.x < 64) {
    int poll = 0;
    const int polls = few_args().polls;
    const uint32_t* first = counter + (size_t)(blockIdx.x % n) * kLine;
    for (; get32(first) == 0 && poll < polls; ++poll) __builtin_amdgcn_s_sleep(36);
    for (;; ++poll) {
      const uint32_t v = lane < n ? get32(counter + (size_t)lane * kLine) : want;
      if (__builtin_amdgcn_ballot_w64(v != want) == 0) break;
      if (poll >= polls) { sh->stop = 1; break; }
    }
  }
  barrier();
  return !__builtin_amdgcn_readfirstlane(sh->stop);
}
// ... for the n tiles of a phase counted on eight counters
__device__ __forceinline__ bool few_wait_phase(const uint32_t* counter, int n, FewShared* sh) {
  return few_wait(counter, min(n, 8), (uint32_t)((n - (threadIdx.x & 63) + 7) / 8), sh);
}
// This tile's stores are behind the caches: counts it as done.  Ends with every wave past its reads of LDS.
__device__ __forceinline__ void few_done(uint32_t* counter) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  barrier();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bf16x8 few_load(__amdgpu_buffer_rsrc_t r, int off, int step) {      // 32 contraction values of 16 rows
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off, step * 2048, 0));
}

__device__ __forceinline__ int few_cached(const FewArgs& a, int r) { return a.pos.kv_len ? a.pos.kv_len[r >> 1] : a.pos.kv_base; }   // cached length

// Tile (row-block mt, column tile nt) of A W^T, 32 rows x CN * 16 columns of W.  PH says what becomes of it.  wait: called when the weights
// are asked for; what it waits for are the tiles that wrote A.
//   16 x 16 x 32 products; a wave takes 1/8 of the contraction.  Its weights are asked for NS steps of 32 ahead (for the usual widths that is
//   all of them), its part of A, which may be asked for only after the wait, NA steps ahead.  No request goes past a wave's last step.
//   DH: head size (q/k/v).  SCALED: A is a row's residual values, un-normalised; its RMSNorm factor multiplies the result.  PH_PART: share `share` of
//   kWideShares of the contraction, whose sums go to a.part.  RB: row-blocks of the tile, mt counts such tiles; they share the weights' registers, and their
//   sums go through LDS one after the other.
template <int PH, int CN, int NS, int NA, int DH = 64, bool SCALED = PH == PH_QKV || PH == PH_GU, int RB = 1, typename Wait>
__device__ __forceinline__ bool few_tile(const FewArgs& a, const bf16_t* A, const bf16_t* W, int K, int mt, int nt, const float* ss, float* ss_out,
                                         bf16_t* out, const float* g_next, int l, float* red, FewShared* sh, uint32_t* done, Wait wait, int share = 0) {
  constexpr int CW = PH == PH_GU ? CN * 8 : CN * 16, CPT = PH == PH_GU ? 2 : CW / 16;       // columns of the result, neighbouring ones per thread
  constexpr int LDC = CN * 16 + 4, WS = 32 * LDC;                  // row and wave stride of the partial sums
  static_assert(NS % NA == 0 && (CPT == 2 || CPT == 4), "");
  const int tid = few_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KB = K >> 4, all = K >> 5, of_share = PH == PH_PART ? (all + kWideShares - 1) / kWideShares : all;
  const int s_first = min(share * of_share, all), s_end = min(s_first + of_share, all);
  const int per = (of_share + kWaves - 1) / kWaves, s0 = min(s_first + wave * per, s_end), n = min(per, s_end - s0);
  const int i16 = lane & 15, g = lane >> 4;
  __amdgpu_buffer_rsrc_t ra[RB];           // (row-blocks past the last repeat it)
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
    ra[rb] = __builtin_amdgcn_make_buffer_rsrc((void*)(A + ((size_t)(RB > 1 ? min(mt * RB + rb, a.MT - 1) : mt) * KB + 2 * s0) * 512), 0, n * 2048, 0x00020000);
  // 16-column groups of W.  Gate/up: the gate columns of CN / 2 groups of hidden units, then their up columns; both stand in blocks of 32,
  // alternating; groups past the end repeat the last
  int group[CN];
#pragma unroll
  for (int t = 0; t < CN; ++t) {
    const int h = min(nt * (CN / 2) + t % (CN / 2), (a.F >> 4) - 1);
    group[t] = PH == PH_GU ? (h >> 1) * 4 + (h & 1) + (t < CN / 2 ? 0 : 2) : nt * CN + t;
  }
  __amdgpu_buffer_rsrc_t rw[CN];
#pragma unroll
  for (int t = 0; t < CN; ++t)
    rw[t] = __builtin_amdgcn_make_buffer_rsrc((void*)(W + ((size_t)(group[t] >> 1) * KB + 2 * s0) * 512 + (group[t] & 1) * 128), 0, n * 2048, 0x00020000);
  // lane l supplies row l % 16 (+ 16: the block's second half) and the contraction values 8 (l / 16) .. + 7 of a step of two blocks
  const int off = (g >> 1) * 1024 + (i16 + 32 * (g & 1)) * 16;
  bf16x8 fw[NS][CN], fa[NA][2 * RB];
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (i < n) {
#pragma unroll
      for (int t = 0; t < CN; ++t) fw[i][t] = few_load(rw[t], off, i);
    }
  auto request = [&](int i, int step) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      fa[i][2 * rb] = few_load(ra[rb], off, step);
      fa[i][2 * rb + 1] = few_load(ra[rb], off + 256, step);
    }
  };
  // this thread's part of the result: CPT neighbouring columns of a row (v: of a column's rows) in each row-block
  const int row = tid >> 4, c0 = (tid & 15) * CPT;
  int base = mt * RB * 32, m = base + row, mc = min(m, a.M - 1);   // of the row-block that is at hand
  const int n0 = nt * CW;                                          // first column
  const int sec = PH == PH_QKV ? n0 / a.d : 0, hd = PH == PH_QKV ? (n0 - sec * a.d) / DH : 0;      // a q/k/v tile is a head's q, k or v, or half of it
  const int e0 = DH == 64 ? 0 : n0 % DH;                           // its first dimension of the head
  float4 cs;
  int slot[4] = {0, 0, 0, 0}, rr[4] = {0, 0, 0, 0};
  auto position = [&] {
    if (sec < 2) {
      const int r = mc / a.T, t = mc - r * a.T;
      rr[0] = r;
      int img;
      token_pos(a.pos, a.tree, r, t, &slot[0], &img);
      cs = make_float4(1.f, 0.f, 1.f, 0.f);
      if (img >= 0) {
        const int gr = min(img / a.pos.grid_w, a.rope_pos - 1), gc = img % a.pos.grid_w;
        constexpr int HALF = DH / 2;
        cs = *(const float4*)(a.rope + ((size_t)(e0 + c0 >= HALF ? gc : gr) * (HALF / 2) + (((e0 + c0) & (HALF - 1)) >> 1)) * 2);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int mv = min(base + (tid & 7) * 4 + i, a.M - 1), r = mv / a.T;
        rr[i] = r;
        slot[i] = few_cached(a, r) + a.tree.first + mv - r * a.T;
      }
    }
  };
  if constexpr (PH == PH_QKV) {
    static_assert(CW == 64, "one head");
    position();
  }
  if (!wait()) return false;
#pragma unroll
  for (int i = 0; i < NA; ++i)
    if (i < n) request(i, i);
  __builtin_amdgcn_sched_barrier(0);
  // inputs of the epilogue, behind the operands
  float xv[CPT], gv[CPT], sq[3] = {0.f, 0.f, 0.f};
  if constexpr (PH == PH_O || PH == PH_DOWN) {
#pragma unroll
    for (int i = 0; i < CPT; i += 2) {
      const float2 v = get2(a.x + (size_t)mc * a.d + n0 + c0 + i);
      xv[i] = v.x;
      xv[i + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int i = 0; i < CPT; ++i) xv[i] = 0.f;
  }
  if constexpr (PH == PH_O || PH == PH_DOWN || PH == PH_INPUT) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) gv[i] = g_next[n0 + c0 + i];
  }
  if constexpr (SCALED) {
#pragma unroll
    for (int i = 0; i < 3; ++i)            // 48 slabs: d 1536; wider rows: the rest in the epilogue
      if ((tid & 15) + 16 * i < a.NS) sq[i] = ss[(size_t)mc * a.NS + (tid & 15) + 16 * i];
  }
  __builtin_amdgcn_sched_barrier(0);
  static_assert(RB == 1 || PH == PH_PART || !SCALED && (PH == PH_QKV || PH == PH_GU), "these inputs are asked for once");
  floatx4 acc[2 * RB][CN];
#pragma unroll
  for (int r = 0; r < 2 * RB; ++r)
#pragma unroll
    for (int t = 0; t < CN; ++t) acc[r][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int c = 0; c < n; c += NS) {
#pragma unroll
    for (int i = 0; i < NS; ++i)
      if (c + i < n) {
        // W A^T: a lane holds one row (lane % 16) and, per accumulator, the columns 4 (lane / 16) .. + 3
#pragma unroll
        for (int r = 0; r < 2 * RB; ++r)
#pragma unroll
          for (int t = 0; t < CN; ++t) acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i][t], fa[i % NA][r], acc[r][t], 0, 0, 0);
        if (c + i + NA < n) request(i % NA, c + i + NA);
        if (c + i + NS < n) {
#pragma unroll
          for (int t = 0; t < CN; ++t) fw[i][t] = few_load(rw[t], off, c + i + NS);
        }
      }
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    if (rb) {
      base += 32;
      m += 32;
      mc = min(m, a.M - 1);
      if constexpr (PH == PH_QKV) position();
      barrier();                             // the sums of the row-block before are read
    }
    {
      float* mine = red + (size_t)wave * WS + i16 * LDC + 4 * g;
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < CN; ++t) *(floatx4*)(mine + r * 16 * LDC + t * 16) = acc[2 * rb + r][t];
    }
    barrier();
    auto sum = [&](const float* p, float (&v)[CPT]) {       // the partial sums of this thread's columns, in a fixed order
      typedef float vec __attribute__((ext_vector_type(CPT)));
      vec s = *(const vec*)p;
#pragma unroll
      for (int w = 1; w < kWaves; ++w) s += *(const vec*)(p + w * WS);
#pragma unroll
      for (int i = 0; i < CPT; ++i) v[i] = s[i];
    };
    auto sum8 = [](float v) {                // over 8 neighbouring lanes
      v += dpp_move<0x141>(v);
      v += dpp_move<0x4E>(v);
      return v + dpp_move<0xB1>(v);
    };
    float sc = 1.f;                          // RMSNorm row factor of this thread's row
    if constexpr (SCALED) {
      float t = sq[0] + sq[1] + sq[2];
      for (int i = (tid & 15) + 48; i < a.NS; i += 16) t += ss[(size_t)mc * a.NS + i];
      t += dpp_move<0x128>(t);
      sc = 1.0f / sqrtf(sum8(t) / (float)a.d + a.eps);
    }
    float v[CPT];
    sum(red + row * LDC + c0, v);
    if constexpr (PH == PH_GU) {
#pragma unroll
      for (int c = c0; c < CW; c += 32) {    // two hidden units, 32 further on two more
        float up[CPT];
        if (c != c0) sum(red + row * LDC + c, v);
        sum(red + row * LDC + CW + c, up);
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
          const float gate = v[i] * sc;
          if (!SCALED && a.exact_gate) v[i] = gate / (1.0f + expf(-gate)) * up[i];
          else v[i] = gate * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gate)) * (up[i] * sc);
        }
        if (m < a.M && n0 + c < a.F) put32(out + pack_index(m, n0 + c, a.F), pack2bf(v[0], v[1]));
      }
    } else if constexpr (PH == PH_QKV) {
#pragma unroll
      for (int i = 0; i < CPT; ++i) v[i] *= sc;
      if (sec < 2) {
        const uint32_t lo = pack2bf(v[0] * cs.x - v[1] * cs.y, v[0] * cs.y + v[1] * cs.x), hi = pack2bf(v[2] * cs.z - v[3] * cs.w, v[2] * cs.w + v[3] * cs.z);
        if (m < a.M) {
          if (sec == 0) put64(out + (size_t)m * a.d + n0 + c0, lo, hi);
          else if (slot[0] >= 0 && slot[0] < a.S_cap) put64(a.kc + a.kv_layer * l + rr[0] * a.kv_row + hd * a.kv_head + k_index(slot[0], e0 + c0, DH), lo, hi);
        }
      } else {
        // v: the 8 slots of a dim are contiguous, so neighbouring lanes take the rows of a dim
        *(float4*)(red + row * LDC + c0) = make_float4(v[0], v[1], v[2], v[3]);      // (this thread's own first partial sums)
        barrier();
        const int col = tid >> 3, r0 = (tid & 7) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (base + r0 + i < a.M && slot[i] >= 0 && slot[i] < a.S_cap)
            put(a.vc + a.kv_layer * l + rr[i] * a.kv_row + hd * a.kv_head + v_index(slot[i], e0 + col, DH), f2bf(red[(r0 + i) * LDC + col]));
      }
    } else if constexpr (PH == PH_PART) {
      if (m < a.M) {
        float* p = a.part + ((size_t)share * a.M + m) * a.d + n0 + c0;
#pragma unroll
        for (int i = 0; i < CPT; i += 2) put64(p + i, __float_as_uint(v[i]), __float_as_uint(v[i + 1]));
      }
    } else {
      float s2 = 0.f;
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        v[i] += xv[i];
        s2 += v[i] * v[i];
      }
      s2 = sum8(s2);
      if (CPT == 2) s2 += dpp_move<0x128>(s2);                       // a slab of the sums of squares: 32 columns
      if (m < a.M) {
#pragma unroll
        for (int i = 0; i < CPT; i += 2) put64(a.x + (size_t)m * a.d + n0 + c0 + i, __float_as_uint(v[i]), __float_as_uint(v[i + 1]));
        bf16_t* o = out + pack_index(m, n0 + c0, a.d);
        if constexpr (CPT == 4) put64(o, pack2bf(v[0] * gv[0], v[1] * gv[1]), pack2bf(v[2] * gv[2], v[3] * gv[3]));
        else put32(o, pack2bf(v[0] * gv[0], v[1] * gv[1]));
        static_assert(kSlab == 32, "");
        if ((c0 & 31) == 0) {
          float* so = ss_out + (size_t)m * a.NS + (n0 + c0) / kSlab;
          put(so, s2);
          if (n0 + c0 + kSlab == a.d)                                // the row's padding
            for (int i = a.d / kSlab; i < a.NS; ++i) put(++so, 0.f);
        }
      }
    }
  }
  few_done(done);
  return true;
}

// Attention of head hd, queries q0 .. q0 + 16 NQB - 1 of rows r0 .. r0 + 8 / NW - 1 (those there are): see k_attn_mfma.  NW waves to a row, which
// take 32-key steps round-robin; steps that lie below the cached length are asked for before the wait.
template <int NQB, int NW, int DH = 64, typename Wait>
__device__ __forceinline__ bool few_attention(const FewArgs& a, const FewBuf& b, int hd, int r0, int q0, int l, float* red, FewShared* sh, uint32_t* done, Wait wait) {
  constexpr int KD = DH / 32, DT = DH / 16, NQ = NQB * 16, PD = DH > 64 ? 1 : 2;
  constexpr int LDO = DH + 4;
  float* s_o = red;                        // [8 waves][NQ][LDO]
  float* s_m = s_o + kWaves * NQ * LDO;
  float* s_l = s_m + kWaves * NQ;
  const int tid = few_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), aw = wave % NW;
  const int r = min(r0 + wave / NW, a.R - 1);        // (past the last row: its work once more, not stored)
  const int g = lane >> 4, ql = lane & 15, T = a.T;
  const int S = few_cached(a, r), n_keys = S + a.tree.first + T, nsteps = min((n_keys + 31) >> 5, a.S_cap >> 5);
  const bf16_t* kb = a.kc + a.kv_layer * l + r * a.kv_row + hd * a.kv_head;
  const bf16_t* vb = a.vc + a.kv_layer * l + r * a.kv_row + hd * a.kv_head;
  bf16x8 kf[PD][2][KD], vf[PD][DT];
  bool early[PD];
#pragma unroll
  for (int p = 0; p < PD; ++p) {
    early[p] = aw + p * NW < min(S >> 5, nsteps);     // wholly below the cached length: nobody writes there
    if (early[p]) VVS_ATTN_LOAD(aw + p * NW, kf[p], vf[p]);
  }
  if (!wait()) return false;
  bf16x8 qf[NQB][KD];
  uint64_t mask[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int tq = min(q0 + qb * 16 + ql, T - 1);      // query rows past T repeat row T - 1 and are not stored
    mask[qb] = a.tree.anc[a.tree.first + tq];
#pragma unroll
    for (int kd = 0; kd < KD; ++kd) qf[qb][kd] = as_bf16x8(*(const uint4*)(b.q + (size_t)(r * T + tq) * a.d + hd * DH + kd * 32 + g * 8));
  }
#pragma unroll
  for (int p = 0; p < PD; ++p)
    if (!early[p] && aw + p * NW < nsteps) VVS_ATTN_LOAD(aw + p * NW, kf[p], vf[p]);
  float m_run[NQB], l_run[NQB];
  floatx4 o[NQB][DT];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    m_run[qb] = -INFINITY;
    l_run[qb] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[qb][dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  for (int base = aw; base < nsteps; base += NW * PD) {
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      const int step = base + p * NW;
      if (step < nsteps) {
        const int key0 = step << 5;
        attn_step<NQB, KD, DT>(kf[p], vf[p], qf, mask, m_run, l_run, o, key0, S, n_keys, key0 + 32 > S, g, a.c_exp);
      }
      if (step + PD * NW < nsteps) VVS_ATTN_LOAD(step + PD * NW, kf[p], vf[p]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int ui = wave * NQ + qb * 16 + ql;
    if (g == 0) { s_m[ui] = m_run[qb]; s_l[ui] = l_run[qb]; }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      *(floatx4*)(s_o + ui * LDO + dt * 16 + 4 * g) = o[qb][dt];
  }
  barrier();
  // wave aw of a row merges its 16-query, 16-dim blocks aw, aw + NW, ...
  for (int blk = aw; blk < NQB * DT; blk += NW) {
    const int qi = (blk / DT) * 16 + ql, dt = blk % DT, w0 = wave - aw;
    float mw[NW], mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) { mw[w] = s_m[(w0 + w) * NQ + qi]; mx = fmaxf(mx, mw[w]); }
    const float m_safe = mx == -INFINITY ? 0.f : mx;
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {         // fixed order
      const float wt = exp2f((mw[w] - m_safe) * a.c_exp);
      sum += s_l[(w0 + w) * NQ + qi] * wt;
      v += *(const floatx4*)(s_o + ((w0 + w) * NQ + qi) * LDO + dt * 16 + 4 * g) * wt;
    }
    const float inv = 1.0f / sum;
    if (q0 + qi < T && r0 + wave / NW < a.R)
      put64(b.att + pack_index(r * T + q0 + qi, hd * DH + dt * 16 + 4 * g, a.d), pack2bf(v[0] * inv, v[1] * inv), pack2bf(v[2] * inv, v[3] * inv));
  }
  few_done(done);
  return true;
}

// LDS: partial sums of gate/up (6 groups of 16 columns), the attention's merge buffers.  More than half of what a CU has, which leaves one workgroup per CU
constexpr size_t kFewLds = sizeof(float) * kWaves * 32 * (6 * 16 + 4);
static_assert(kFewLds >= sizeof(float) * kWaves * 32 * (68 + 2) && kFewLds > 80 * 1024, "");

// How the tiles are dealt: 1 where all workgroups are there, 2 where they are not within the bounded time; the same answer for all.  They are counted
// on eight counters (256 atomics on one take 3 us) and the first workgroup tells the others.  (Not inlined: that doubles the scalar registers that
// the tile loop spills, 2 % of its time.)
__device__ __attribute__((noinline)) int few_dealing(uint32_t* sync, int id) {
  __hip_atomic_fetch_add(sync + (3 + (id & 7)) * kLine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t mode = 0;
  const long t0 = wall_clock64();
  do {
    uint32_t verdict = wall_clock64() - t0 > kAdmission ? 2u : 0u, here = 0;
    if (id == 0) {
      for (int i = 0; i < 8; ++i) here += get32(sync + (3 + i) * kLine);
      if (here == kGroups) verdict = 1;
    }
    if (verdict) __hip_atomic_compare_exchange_strong(sync, &mode, verdict, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    mode = get32(sync);
  } while (mode == 0);
  return (int)mode;
}

// The last workgroup notes whether all tiles were computed, and leaves the counters as it found them: zero
__device__ __forceinline__ void few_leave(FewShared* sh) {
  const FewArgs& e = few_args();
  barrier();
  if (threadIdx.x == 0) {
    auto last = [](uint32_t* counter, uint32_t n) { return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1; };
    uint32_t* stopped = e.sync + 2 * kLine + 1;
    if (sh->stop) {
      __hip_atomic_fetch_add(stopped, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // ... before this workgroup counts as done
    }
    sh->last = last(e.sync + (11 + (blockIdx.x & 7)) * kLine, kGroups / 8) && last(e.sync + 2 * kLine, 8);
    if (sh->last) {
      const uint32_t n = get32(stopped);
      *e.gave_up = e.fc ? *e.gave_up | n : n;
    }
  }
  barrier();
  if (sh->last)
    for (size_t i = threadIdx.x; i < (kFewHead + (size_t)few_layer_counters(e.H, e.MT) * e.L + 8) * kLine / 4; i += kThreads) ((uint4*)e.sync)[i] = make_uint4(0, 0, 0, 0);
}

template <int NQB>
__global__ __launch_bounds__(kThreads, 2) void k_layers_few(const FewArgs args) {
  extern __shared__ float red[];
  __shared__ FewShared sh;
  uint32_t* sync = few_args().sync;
  if (threadIdx.x == 0) {
    sh.stop = 0;
    sh.mode = few_dealing(sync, blockIdx.x);
  }
  barrier();
  const bool dealt = __builtin_amdgcn_readfirstlane(sh.mode) == 1;
  for (int tk = blockIdx.x;; tk += kGroups) {
    if (!dealt) {
      uint32_t* next = few_args().sync + kLine;
      if (threadIdx.x == 0) sh.ticket = (int)__hip_atomic_fetch_add(next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      barrier();
      tk = sh.ticket;
      barrier();
    }
    tk = __builtin_amdgcn_readfirstlane(tk);
    const FewArgs& a = few_args();
    const int d = a.d, MT = a.MT;
    const int n_o = MT * (d >> 6), n_qkv = 3 * n_o, per_row = (a.T + 16 * NQB - 1) / (16 * NQB), row_groups = (a.R + a.rows_per_unit - 1) / a.rows_per_unit, n_att = a.H * row_groups * per_row, gu_tiles = (a.F + 47) / 48, n_gu = MT * gu_tiles, n_down = MT * (d >> 5);
    const int n_in = a.fc ? n_down : 0, per_layer = n_qkv + n_att + n_o + n_gu + n_down, total = n_in + per_layer * a.L;
    uint32_t* counters = a.sync + kFewHead * kLine;
    const int lc = few_layer_counters(a.H, MT);
    if (tk >= total) break;
    bool ok;
    if (tk < n_in) {                       // x = [embedding ; feature] W_fc, counted as the phase in front of layer 0
      int mt, nt;
      tile_of(tk, MT, d >> 5, &mt, &nt);
      ok = few_tile<PH_INPUT, 2, 14, 7>(a, a.din, a.fc, 2 * d, mt, nt, nullptr, a.ss, a.xb, (const float*)(a.layer0 + a.o_g1), 0, red, &sh,
                                        counters + ((size_t)lc * a.L + (tk & 7)) * kLine, [] { return true; });
    } else {
      const int l = (tk - n_in) / per_layer;
      int j = tk - n_in - l * per_layer;
      const char* lw = a.layer0 + a.layer_stride * l;
      uint32_t* ch = counters + (size_t)lc * l * kLine;              // q/k/v: [head][row tile]
      uint32_t* cp = ch + (size_t)a.H * MT * kLine;                  // attention, O, gate/up, down: 8 each
      const FewBuf b = few_buf(a, l);
      int mt, nt;
      if (j < n_qkv) {
        const bf16_t* A = a.xb;
        const float* ss = a.ss;
        if (l) {
          const FewBuf p = few_buf(a, l - 1);
          A = p.xb1;
          ss = p.ss1;
        }
        tile_of(j, MT, 3 * d >> 6, &mt, &nt);
        const uint32_t* before = l ? cp - (size_t)lc * kLine + 3 * 8 * kLine : counters + (size_t)lc * a.L * kLine;
        ok = few_tile<PH_QKV, 4, 6, 6>(a, A, (const bf16_t*)(lw + a.o_wqkv), d, mt, nt, ss, nullptr, b.q, nullptr, l, red, &sh,
                                        ch + ((size_t)(nt % a.H) * MT + mt) * kLine,
                                        [&] { return l || n_in ? few_wait_phase(before, n_down, &sh) : true; });
      } else if ((j -= n_qkv) < n_att) {
        const int hd = j % a.H, rq = j / a.H, rg = rq / per_row, r0 = rg * a.rows_per_unit, q0 = (rq - rg * per_row) * 16 * NQB;
        const int first = r0 * a.T >> 5, n = ((min(a.M, (r0 + a.rows_per_unit) * a.T) - 1) >> 5) - first + 1;
        auto wait = [&] { return few_wait(ch + ((size_t)hd * MT + first) * kLine, n, 3u, &sh); };
        uint32_t* done = cp + (j & 7) * kLine;
        if (a.rows_per_unit == 1) ok = few_attention<NQB, 8>(a, b, hd, r0, q0, l, red, &sh, done, wait);
        else if (a.rows_per_unit == 2) ok = few_attention<NQB, 4>(a, b, hd, r0, q0, l, red, &sh, done, wait);
        else ok = few_attention<NQB, 2>(a, b, hd, r0, q0, l, red, &sh, done, wait);
      } else if ((j -= n_att) < n_o) {
        tile_of(j, MT, d >> 6, &mt, &nt);
        ok = few_tile<PH_O, 4, 6, 6>(a, b.att, (const bf16_t*)(lw + a.o_wo), d, mt, nt, nullptr, b.ss2, b.xb2, (const float*)(lw + a.o_g2), l, red, &sh,
                                      cp + (8 + (j & 7)) * kLine, [&] { return few_wait_phase(cp, n_att, &sh); });
      } else if ((j -= n_o) < n_gu) {
        tile_of(j, MT, gu_tiles, &mt, &nt);
        ok = few_tile<PH_GU, 6, 5, 5>(a, b.xb2, (const bf16_t*)(lw + a.o_wgu), d, mt, nt, b.ss2, nullptr, b.act, nullptr, l, red, &sh,
                                       cp + (16 + (j & 7)) * kLine, [&] { return few_wait_phase(cp + 8 * kLine, n_o, &sh); });
      } else {
        j -= n_gu;
        const bool last = l + 1 == a.L;
        tile_of(j, MT, d >> 5, &mt, &nt);
        ok = few_tile<PH_DOWN, 2, 14, 7>(a, b.act, (const bf16_t*)(lw + a.o_wd), a.F, mt, nt, nullptr, last ? a.ss : b.ss1, last ? a.xb : b.xb1,
                                         last ? a.gf : (const float*)(lw + a.layer_stride + a.o_g1), l, red, &sh, cp + (24 + (j & 7)) * kLine,
                                         [&] { return few_wait_phase(cp + 16 * kLine, n_gu, &sh); });
      }
    }
    if (!ok) break;
  }
  few_leave(&sh);
}

// Row m: x += the partial sums in front of it (has_part), out = bf16(x / rms * g), in packed order
template <typename Wait>
__device__ __forceinline__ bool few_norm(const FewArgs& a, int m, bool has_part, const float* g, bf16_t* out, float* red, uint32_t* done, Wait wait) {
  const int tid = few_tid(), k0 = min(tid * 8, a.d - 8);
  const bool mine = tid * 8 < a.d;
  const float4 ga = *(const float4*)(g + k0), gb = *(const float4*)(g + k0 + 4);
  if (!wait()) return false;
  float v[8];
  float* xr = a.x + (size_t)m * a.d + k0;
  float2 x2[4], p2[kWideShares][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) x2[i] = get2(xr + 2 * i);
  if (has_part) {
#pragma unroll
    for (int s = 0; s < kWideShares; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) p2[s][i] = get2(a.part + ((size_t)s * a.M + m) * a.d + k0 + 2 * i);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) { v[2 * i] = x2[i].x; v[2 * i + 1] = x2[i].y; }
  if (has_part) {
#pragma unroll
    for (int s = 0; s < kWideShares; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) { v[2 * i] += p2[s][i].x; v[2 * i + 1] += p2[s][i].y; }
    if (mine)
#pragma unroll
      for (int i = 0; i < 4; ++i) put64(xr + 2 * i, __float_as_uint(v[2 * i]), __float_as_uint(v[2 * i + 1]));
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) ss += v[i] * v[i];
  ss = wave_sum(mine ? ss : 0.f);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  barrier();
  float t = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) t += red[w];
  const float scale = 1.0f / sqrtf(t / (float)a.d + a.eps);
  if (mine) {
    bf16_t* o = out + pack_index(m, k0, a.d);
    put64(o, pack2bf(v[0] * scale * ga.x, v[1] * scale * ga.y), pack2bf(v[2] * scale * ga.z, v[3] * scale * ga.w));
    put64(o + 4, pack2bf(v[4] * scale * gb.x, v[5] * scale * gb.y), pack2bf(v[6] * scale * gb.z, v[7] * scale * gb.w));
  }
  few_done(done);
  return true;
}

// The same for wide layers, whose weights stream from HBM and whose norms round their output (plan_fused): normalisations are phases of their own, one
// row to a tile, and O and down leave partial sums of kWideShares shares of the contraction, which the normalisation behind them adds to x.  The last
// layer's are left to the caller.
//   Bound by HBM: 404 MB a layer at d 4096, d_ff 11008.  Launches left it idle at every start and end and for normalisation and attention (23 us of 113);
//   here the weights of a workgroup's next tile, up to 256 KB, are on their way while it waits.  d 4096, 32 layers, 28 rows 3601 -> 3311 us, 2 rows 3406 ->
//   2990 (4.3 TB/s over all).  Where the rest goes (one layer of 105 us, 28 rows): normalisation 10 and 8 us, during which the weights arrive that are asked
//   for ahead; q/k/v 19 (192 tiles: a CU gets 25 GB/s from HBM), attention 10, O 12, gate/up 30 (4.3 TB/s: a quarter of what a CU
//   pulls in are activations), down 18.  Two shares of 32 columns: 4 shares of 64 columns 1 % slower (twice the sums), 8 of 128 5 %.
//   Requested ahead, steps of q/k/v 8, of gate/up 5, of O and down 8: 6 to 16 the same within 1 %, q/k/v all 16 steps (spilled) 18 % slower.
template <int NQB, int DH, int RB>
__global__ __launch_bounds__(kThreads, 2) void k_layers_wide(const FewArgs args) {
  extern __shared__ float red[];
  __shared__ FewShared sh;
  uint32_t* sync = few_args().sync;      // (the head of k_layers_few; as functions that both call it is 0.3 % slower)
  if (threadIdx.x == 0) {
    sh.stop = 0;
    sh.mode = few_dealing(sync, blockIdx.x);
  }
  barrier();
  const bool dealt = __builtin_amdgcn_readfirstlane(sh.mode) == 1;
  for (int tk = blockIdx.x;; tk += kGroups) {
    if (!dealt) {
      uint32_t* next = few_args().sync + kLine;
      if (threadIdx.x == 0) sh.ticket = (int)__hip_atomic_fetch_add(next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      barrier();
      tk = sh.ticket;
      barrier();
    }
    tk = __builtin_amdgcn_readfirstlane(tk);
    const FewArgs& a = few_args();
    const int d = a.d, MT = (a.MT + RB - 1) / RB, n_norm = a.M;
    const int cols = d >> 6, n_qkv = 3 * MT * cols, per_row = (a.T + 16 * NQB - 1) / (16 * NQB), row_groups = (a.R + a.rows_per_unit - 1) / a.rows_per_unit;
    const int n_att = a.H * row_groups * per_row, pcols = d >> 5, n_whole = MT * pcols, n_part = n_whole * kWideShares, gu_tiles = (a.F + 47) / 48, n_gu = MT * gu_tiles;
    const int per_layer = 2 * n_norm + n_qkv + n_att + 2 * n_part + n_gu;
    if (tk >= per_layer * a.L) break;
    const int l = tk / per_layer, lc = few_layer_counters(a.H, a.MT);
    int j = tk - l * per_layer;
    const char* lw = a.layer0 + a.layer_stride * l;
    uint32_t* ch = a.sync + (kFewHead + (size_t)lc * l) * kLine;     // q/k/v: [head][row tile]
    uint32_t* cp = ch + (size_t)a.H * a.MT * kLine;                    // attention, O, gate/up, down, the two norms: 8 each
    const FewBuf b = few_buf(a, l);
    int mt, nt;
    bool ok;
    if (j < n_norm) {
      ok = few_norm(a, j, l > 0, (const float*)(lw + a.o_g1), b.xb1, red, cp + (32 + (j & 7)) * kLine,
                    [&] { return l ? few_wait_phase(cp + (24 - lc) * kLine, n_part, &sh) : true; });
    } else if ((j -= n_norm) < n_qkv) {
      tile_of(j, MT, 3 * cols, &mt, &nt);
      ok = few_tile<PH_QKV, 4, RB == 1 ? 8 : 6, RB == 1 ? 4 : 3, DH, false, RB>(a, b.xb1, (const bf16_t*)(lw + a.o_wqkv), d, mt, nt, nullptr, nullptr, b.q, nullptr, l, red, &sh,
                                                ch + ((size_t)(nt % cols / (DH / 64)) * MT + mt) * kLine,
                                                [&] { return few_wait_phase(cp + 32 * kLine, n_norm, &sh); });
    } else if ((j -= n_qkv) < n_att) {
      const int hd = j % a.H, rq = j / a.H, rg = rq / per_row, r0 = rg * a.rows_per_unit, q0 = (rq - rg * per_row) * 16 * NQB;
      const int first = r0 * a.T / (32 * RB), n = (min(a.M, (r0 + a.rows_per_unit) * a.T) - 1) / (32 * RB) - first + 1;
      auto wait = [&] { return few_wait(ch + ((size_t)hd * MT + first) * kLine, n, 3u * (DH / 64), &sh); };
      uint32_t* done = cp + (j & 7) * kLine;
      if (a.rows_per_unit == 1) ok = few_attention<NQB, 8, DH>(a, b, hd, r0, q0, l, red, &sh, done, wait);
      else if (a.rows_per_unit == 2) ok = few_attention<NQB, 4, DH>(a, b, hd, r0, q0, l, red, &sh, done, wait);
      else ok = few_attention<NQB, 2, DH>(a, b, hd, r0, q0, l, red, &sh, done, wait);
    } else if ((j -= n_att) < n_part) {
      tile_of(j % n_whole, MT, pcols, &mt, &nt);
      ok = few_tile<PH_PART, 2, 8, RB == 1 ? 8 : 4, 64, false, RB>(a, b.att, (const bf16_t*)(lw + a.o_wo), d, mt, nt, nullptr, nullptr, nullptr, nullptr, l, red, &sh,
                                      cp + (8 + (j & 7)) * kLine, [&] { return few_wait_phase(cp, n_att, &sh); }, j / n_whole);
    } else if ((j -= n_part) < n_norm) {
      ok = few_norm(a, j, true, (const float*)(lw + a.o_g2), b.xb2, red, cp + (40 + (j & 7)) * kLine,
                    [&] { return few_wait_phase(cp + 8 * kLine, n_part, &sh); });
    } else if ((j -= n_norm) < n_gu) {
      tile_of(j, MT, gu_tiles, &mt, &nt);
      ok = few_tile<PH_GU, 6, RB == 1 ? 5 : 3, RB == 1 ? 5 : 3, 64, false, RB>(a, b.xb2, (const bf16_t*)(lw + a.o_wgu), d, mt, nt, nullptr, nullptr, b.act, nullptr, l, red, &sh,
                                               cp + (16 + (j & 7)) * kLine, [&] { return few_wait_phase(cp + 40 * kLine, n_norm, &sh); });
    } else {
      j -= n_gu;
      tile_of(j % n_whole, MT, pcols, &mt, &nt);
      ok = few_tile<PH_PART, 2, 8, RB == 1 ? 8 : 4, 64, false, RB>(a, b.act, (const bf16_t*)(lw + a.o_wd), a.F, mt, nt, nullptr, nullptr, nullptr, nullptr, l, red, &sh,
                                      cp + (24 + (j & 7)) * kLine, [&] { return few_wait_phase(cp + 16 * kLine, n_gu, &sh); }, j / n_whole);
    }
    if (!ok) break;
  }
  few_leave(&sh);
}
constexpr size_t kWideLds = sizeof(float) * kWaves * 32 * (128 + 4 + 2);

// All layers of a forward of at most few_rows(c) rows and VVS_MAX_T tokens per row.  In: x, its packed operand bf16(x g1) (rows unpadded) and sums of
// squares, or the drafter's input rows.  Out: the same of the last layer, with the gain of the final norm.
static FewArgs few_arguments(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int T, bool from_din) {
  const int M = c->R * T, MT = (M + 31) / 32;
  FewArgs a{};
  a.layer0 = c->pw + c->p.layer0;
  a.layer_stride = c->p.layer_stride;
  a.o_g1 = c->p.g1; a.o_wqkv = c->p.wqkv; a.o_wo = c->p.wo; a.o_g2 = c->p.g2; a.o_wgu = c->p.wgu; a.o_wd = c->p.wd;
  a.gf = (const float*)(c->pw + c->p.gf);
  if (from_din) {
    a.fc = (const bf16_t*)(c->pw + c->p.fc);
    a.din = (const bf16_t*)(c->ws + c->w.din);
  }
  a.x = (float*)(c->ws + c->w.x);
  a.xb = (bf16_t*)(c->ws + c->w.h);
  a.ss = (float*)(c->ws + c->w.ss);
  a.buf = c->ws + c->w.few_buf;
  a.buf_stride = few_buf_bytes(MT * 32, c->d, c->F);
  a.kc = (bf16_t*)c->kv;
  a.vc = (bf16_t*)c->kv + c->kv_v_off;
  a.kv_layer = c->kv_layer_stride; a.kv_row = c->kv_row_stride; a.kv_head = c->kv_head_stride;
  a.rope = (const float*)(c->ws + c->w.rope_tab);
  a.sync = (uint32_t*)(c->ws + c->w.few_sync);
  a.gave_up = (uint32_t*)(c->ws + c->w.few_gave_up);
  a.polls = c->wait_polls;
  a.L = c->L; a.M = M; a.MT = MT; a.T = T; a.d = c->d; a.H = c->H; a.F = c->F; a.R = c->R; a.NS = n_slabs(c->d); a.S_cap = c->S_cap;
  a.rope_pos = c->rope_pos;
  a.eps = c->cfg.rms_eps;
  a.c_exp = 1.4426950408889634f / sqrtf((float)c->dh);
  a.pos = pos;
  a.tree = tree;
  a.part = (float*)(c->ws + c->w.gemm_out);
  return a;
}

void launch_layers_few(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int T, bool from_din, hipStream_t s) {
  FewArgs a = few_arguments(c, tree, pos, T, from_din);
#define VVS_FEW(NQB)                                                                                                            \
  {                                                                                                                             \
    allow_dynamic_lds(reinterpret_cast<const void*>(&k_layers_few<NQB>), kFewLds);                                               \
    hipLaunchKernelGGL((k_layers_few<NQB>), dim3(kGroups), dim3(kThreads), kFewLds, s, a);                                           \
  }
  // attention: 16 queries to a unit while all units of a row's waves run at once, else 32; more units than CUs: rows share one
  const int pairs = c->H * c->R, nqb = pairs * ((T + 15) / 16) <= 192 ? 1 : 2, units = pairs * ((T + 16 * nqb - 1) / (16 * nqb));
  a.rows_per_unit = units <= 256 ? 1 : units <= 512 ? 2 : 4;
  if (T <= 16 || nqb == 1) VVS_FEW(1) else VVS_FEW(2)
#undef VVS_FEW
}

// The same for wide layers, of at most few_wide_rows(c) rows.  In: x.  Out: x of the last layer without its down projection, whose kFewWideShares partial
// sums [M][d] are in gemm_out.
void launch_layers_wide(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int T, hipStream_t s) {
  FewArgs a = few_arguments(c, tree, pos, T, false);
  a.exact_gate = plan_gate_up(c, a.M).splits > 1;
  const int nqb = T <= 16 ? 1 : 2, units = c->H * c->R * ((T + 16 * nqb - 1) / (16 * nqb));
  a.rows_per_unit = units <= 256 ? 1 : units <= 512 ? 2 : 4;
#define VVS_WIDE1(NQB, DH, RB)                                                                                                       \
  {                                                                                                                             \
    allow_dynamic_lds(reinterpret_cast<const void*>(&k_layers_wide<NQB, DH, RB>), kWideLds);                                         \
    hipLaunchKernelGGL((k_layers_wide<NQB, DH, RB>), dim3(kGroups), dim3(kThreads), kWideLds, s, a);                                  \
  }
  // Two row-blocks to a tile read the weights once instead of twice, and leave half as many tiles: from where O and down have more than one for each
  // CU.  us per layer, one / two, 40 and 64 rows: d 1536 40.1 / 49.0, 40.9 / 47.5; 2048 (d_ff 8192) 62.0 / 68.9, 64.7 / 70.2; 2560 86.1 / 77.0, 88.8 /
  // 78.6; 3072 (3072) 81.9 / 76.6, 83.2 / 76.8;  96 and 128 rows, d 1536 55.9 / 52.6, 67.0 / 54.5, 2048 78.0 / 63.6, 82.9 / 69.2.
  const bool two = a.MT > 1 && (a.MT > 2 || c->d > 2048);
#define VVS_WIDE(NQB, DH) { if (two) VVS_WIDE1(NQB, DH, 2) else VVS_WIDE1(NQB, DH, 1) }
  if (c->dh == 64) { if (nqb == 1) VVS_WIDE(1, 64) else VVS_WIDE(2, 64) }
  else { if (nqb == 1) VVS_WIDE(1, 128) else VVS_WIDE(2, 128) }
#undef VVS_WIDE
#undef VVS_WIDE1
}

}  // namespace vvs
