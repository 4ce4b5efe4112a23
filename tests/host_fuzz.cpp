// Host-only exerciser of the library's planner and argument checks, built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_host_sanitized.py.  The HIP runtime and every kernel launcher
// are replaced by host stand-ins (a "device" buffer is ordinary memory of exactly the size vvs_query_sizes
// asked for; fills and copies really touch it), so that the complete call sequences - create, load, prefill,
// verify with and without unverified tokens, commit, draft, path similarity, inspection - run their host
// side under the sanitizers without a GPU, on random valid and invalid inputs.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <array>
#include <random>
#include <thread>
#include <vector>
#include "vvs_internal.h"

// ---- HIP runtime stand-ins (only what the host file uses)
extern "C" {
static int g_cus = 256;
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* dev) { *dev = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_cus; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) { memcpy(dst, src, n); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
}

// ---- launcher stand-ins: no arithmetic; the ones that have a size touch their buffers
namespace vvs {
static long g_launches = 0;
static DraftLevel g_level;                                      // of the drafting call under way
static bool g_draft_begins = false;
void launch_fill_zero(void* p, size_t bytes, hipStream_t) { memset(p, 0, bytes); ++g_launches; }
void launch_copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t) { memmove(dst, src, bytes); ++g_launches; }
void launch_fill_probe(const void*, size_t, size_t, int, int, int, int, uint32_t*, hipStream_t) { ++g_launches; }
void launch_pack_weights(Ctx*, const void* const*, hipStream_t) { ++g_launches; }
void launch_forward(Ctx* c, const TreeDesc& tree, const PosDesc& pos, int T, const int32_t*, const void*, const void*, int, const int32_t*, int,
                    int, hipStream_t, bool from_din) {
  if (T < 1 || T > c->Tmax && T > c->chunk) abort();            // a forward never exceeds what the workspace was sized for
  if (tree.T != T) abort();
  // a drafting level is a forward of its new tokens in the block's slots and logit rows; every other call is one of all tokens in rows of its own
  if (from_din ? tree.first != g_level.first || tree.all != g_level.all || T != g_level.Tq : tree.first || tree.all) abort();
  for (int t = 0; t < T; ++t)
    if (!((tree.anc[t] >> t) & 1ull) || (t && tree.parent[t] >= t)) abort();
  memset(c->ws + c->w.x, 0, sizeof(float) * (size_t)c->R * T * c->d);
  // a verify or drafting call may lay its normalised operand out with 32 or 64 rows per row; gemm_out is the next buffer
  const size_t rows = (size_t)c->R * (pos.kv_len && c->esz == 2 ? (T <= 32 ? 32 : 64) : T);
  if (rows * c->d * c->esz > c->w.gemm_out - c->w.h) abort();
  if (from_din) memset(c->ws + c->w.din, 0, c->esz * (size_t)c->R * T * 2 * c->d);
  ++g_launches;
}
void launch_build_tokens(Ctx* c, int T, const int32_t*, hipStream_t) { memset(c->ws + c->w.tokens, 0, sizeof(int32_t) * c->B * T); ++g_launches; }
void launch_accept(Ctx*, const TreeDesc&, int, const float*, const int32_t*, const float*, const float*, int, int, int, int, int, bool, int32_t*,
                   int32_t*, int32_t*, bool, const uint32_t*, hipStream_t) { ++g_launches; }
vvs_status launch_accept_noalloc(Ctx*, const TreeDesc&, int, const float*, const int32_t*, const float*, const float*, int, int32_t*, int32_t*,
                                 int32_t*, hipStream_t, std::string*) { ++g_launches; return VVS_OK; }
void launch_prefill_finish(Ctx*, int, int32_t*, hipStream_t) { ++g_launches; }
void launch_commit(Ctx*, hipStream_t) { ++g_launches; }
void launch_push_prefill_feature(Ctx*, int, hipStream_t) { ++g_launches; }
void launch_read_features(Ctx*, float*, int32_t*, hipStream_t) { ++g_launches; }
void launch_path_similarity(Ctx*, const TreeDesc&, int, const int32_t*, float, int, float*, hipStream_t) { ++g_launches; }
void launch_read_state(Ctx*, int32_t*, hipStream_t) { ++g_launches; }
void launch_set_state(Ctx*, const int32_t*, hipStream_t) { ++g_launches; }
void launch_debug_logits(Ctx*, float*, float*, float*, hipStream_t) { ++g_launches; }
void launch_debug_kv(Ctx*, int, int, int, float*, float*, hipStream_t) { ++g_launches; }
void launch_debug_gemm(Ctx*, int, int, int, const void*, const void*, void*, float*, hipStream_t) { ++g_launches; }
void launch_draft_state(Ctx*, const Ctx*, int, int, hipStream_t) { g_draft_begins = true; ++g_launches; }
void launch_draft_zero_leaves(Ctx*, const TreeDesc&, float*, hipStream_t) { ++g_launches; }
void launch_draft_input(Ctx* dr, const Ctx*, const DraftLevel& lv, const int32_t*, const int32_t*, hipStream_t) {
  if (lv.Tq < lv.k || lv.Tq > dr->Tmax) abort();
  // level 0 brings the pairs; every further one what follows the tokens so far, whose parents are among the new ones of the level before (the
  // input rows are read from its residual stream, which holds no others)
  if (lv.first >= lv.Tq || lv.Tq > lv.all || lv.all > dr->Tmax) abort();
  if (g_draft_begins ? lv.first != 0 || lv.Tq != lv.k : lv.first != lv.Tq_prev || lv.first_prev != g_level.first || lv.Tq_prev != g_level.Tq || lv.all != g_level.all) abort();
  for (int t = std::max(lv.k, lv.first); t < lv.Tq; ++t)
    if (lv.node[t] < 1 || lv.node[t] > lv.n_nodes || lv.parent_slot[t] < lv.k - 1 || lv.parent_slot[t] < lv.first_prev || lv.parent_slot[t] >= lv.Tq_prev) abort();
  g_level = lv;
  g_draft_begins = false;
  ++g_launches;
}
void launch_draft_select(Ctx*, const DraftLevel& lv, const TreeDesc& shape, const int32_t*, int32_t*, float*, hipStream_t) {
  for (int i = 0; i < lv.n_sel; ++i)                            // (this level's logits)
    if (lv.sel_slot[i] < lv.k - 1 || lv.sel_slot[i] < lv.first || lv.sel_slot[i] >= lv.Tq || shape.first_child[lv.sel_node[i]] < 0) abort();
  ++g_launches;
}
}  // namespace vvs

static std::mt19937 rng(12345);
static int ri(int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); }

static vvs_config base_config(bool bf16, bool drafter) {
  vvs_config c;
  memset(&c, 0, sizeof(c));
  c.n_layers = drafter ? 1 : 2; c.d_model = bf16 ? 256 : 64; c.n_heads = 4; c.d_ff = bf16 ? 512 : 96; c.vocab = 512;
  c.logit_lo = bf16 ? 64 : 0; c.logit_hi = bf16 ? 64 + 256 : 512; c.grid_h = 6; c.grid_w = 5; c.prefix_len = 3;
  c.prefix_kind = VVS_PREFIX_CLASS; c.n_classes = 10; c.n_prompts = 3; c.max_nodes = 40; c.dtype = bf16 ? VVS_BF16 : VVS_FP32;
  c.cfg_scale = 3.f; c.rms_eps = 1e-5f; c.rope_base = 10000.f; c.relax_k = 0; c.relax_delta = 0.f;
  c.feature_slots = drafter ? 0 : 5; c.feature_pre_norm = 0; c.draft_input = drafter ? 1 : 0;
  return c;
}

struct Dev {   // the three "device" buffers of a context, exactly as large as asked for
  std::vector<char> kv, ws, pw;
  char *akv, *aws, *apw;
  void alloc(const vvs_config& c) {
    size_t a, b, d;
    if (vvs_query_sizes(&c, &a, &b, &d) != VVS_OK) { printf("query_sizes failed: %s\n", vvs_last_error(nullptr)); exit(1); }
    kv.resize(a + 256); ws.resize(b + 256); pw.resize(d + 256);
    akv = (char*)(((uintptr_t)kv.data() + 255) & ~(uintptr_t)255);
    aws = (char*)(((uintptr_t)ws.data() + 255) & ~(uintptr_t)255);
    apw = (char*)(((uintptr_t)pw.data() + 255) & ~(uintptr_t)255);
    // shrink to the exact size so that a write past the end is caught: copies with no slack behind the aligned start
    kv.resize((akv - kv.data()) + a); ws.resize((aws - ws.data()) + b); pw.resize((apw - pw.data()) + d);
    akv = (char*)(((uintptr_t)kv.data() + 255) & ~(uintptr_t)255);
    aws = (char*)(((uintptr_t)ws.data() + 255) & ~(uintptr_t)255);
    apw = (char*)(((uintptr_t)pw.data() + 255) & ~(uintptr_t)255);
  }
};

static void random_tree(int n, std::vector<int32_t>& parent, bool valid) {
  parent.resize(n > 0 ? n : 1);
  for (int j = 1; j <= n; ++j) parent[j - 1] = valid ? ri(0, j - 1) : ri(-2, j + 2);
}

// `host_fuzz plans`: for every line "partial N K M", "qkv d F M" or "gate_up d F M" on the standard input the tile and the shares of that launch
static int print_plans() {
  vvs_config cfg = base_config(true, false);
  vvs::Ctx c;
  std::string err;
  if (vvs::plan_sizes(&cfg, &c, &err) != VVS_OK) return 1;
  char kind[16];
  for (int a, b, m; scanf("%15s %d %d %d", kind, &a, &b, &m) == 4;) {
    c.d = a;
    c.F = b;
    const vvs::GemmPlan p = !strcmp(kind, "partial") ? vvs::plan_partial(&c, m, a, b) : !strcmp(kind, "qkv") ? vvs::plan_qkv(&c, m) : vvs::plan_gate_up(&c, m);
    printf("%d %d %d %d\n", p.bm, p.bn, p.splits, (int)p.shared);
  }
  return 0;
}

// `host_fuzz threads`, built with ThreadSanitizer: what contexts on different threads share
static int run_threads() {
  std::vector<std::thread> all;
  for (int t = 0; t < 4; ++t)
    all.emplace_back([t] {
      for (int i = 0; i < 2000; ++i) vvs::allow_dynamic_lds((const void*)(uintptr_t)(1 + (i * (t + 1)) % 97), 1 << 17);
    });
  for (auto& t : all) t.join();
  printf("threads ok\n");
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 1 && !strcmp(argv[1], "threads")) return run_threads();
  if (argc > 1 && !strcmp(argv[1], "plans")) return print_plans();
  // 1. topology checks and the verification-free step on random input, valid and not
  for (int it = 0; it < 4000; ++it) {
    const int n = ri(-2, 70);
    std::vector<int32_t> parent;
    const bool valid = it % 3 != 0;
    random_tree(n, parent, valid);
    int32_t depth[VVS_MAX_T + 8], pout[VVS_MAX_T + 8], nodes[VVS_MAX_T], kept = -1;
    vvs_status st = vvs_check_tree(n, n > 0 ? parent.data() : nullptr, nullptr, depth, pout);
    if (valid && n >= 0 && n <= VVS_MAX_T - 1 && st != VVS_OK) { printf("valid tree refused (n %d)\n", n); return 1; }
    if ((n < 0 || n > VVS_MAX_T - 1) && st == VVS_OK) { printf("n %d accepted\n", n); return 1; }
    if (st == VVS_OK && n > 0) {
      const int T = n + 1;
      std::vector<uint8_t> mask((size_t)T * T, 0);
      for (int i = 0; i < T; ++i) { int j = i; for (;;) { mask[(size_t)i * T + j] = 1; if (!j) break; j = pout[j - 1]; } }
      if (vvs_check_tree(n, nullptr, mask.data(), depth, pout) != VVS_OK) { printf("own mask refused\n"); return 1; }
      if (vvs_check_tree(n, parent.data(), mask.data(), nullptr, nullptr) != VVS_OK) { printf("parent + mask refused\n"); return 1; }
      mask[(size_t)ri(1, n) * T] = 0;                         // a node that no longer sees the root
      if (vvs_check_tree(n, nullptr, mask.data(), nullptr, nullptr) == VVS_OK) { printf("broken mask accepted\n"); return 1; }
      const float u = it % 7 == 0 ? 1.0f : (float)(rng() % 1000) / 1000.f;
      st = vvs_select_unverified(n, parent.data(), nullptr, u, nodes, &kept);
      if (u >= 1.0f) {                                        // the uniform must lie in [0, 1)
        if (st != VVS_EINVAL) { printf("select_unverified accepted u = 1\n"); return 1; }
        continue;
      }
      if (st != VVS_OK || kept < 1 || kept > n) { printf("select_unverified: status %d kept %d\n", st, kept); return 1; }
      for (int i = 0; i < kept; ++i)
        if (nodes[i] < 1 || nodes[i] > n || (i ? pout[nodes[i] - 1] != nodes[i - 1] : pout[nodes[i] - 1] != 0)) { printf("kept path is not a path\n"); return 1; }
    }
    (void)vvs_skip_uniform(ri(-3, 50), ri(-2, 6));
    (void)vvs_skip_dynamic((float)ri(-5, 15) / 10.f, 0.7f, ri(0, 1));
  }
  // 2. size queries on random configurations never crash and refuse what they cannot serve
  for (int it = 0; it < 2000; ++it) {
    vvs_config c = base_config(it & 1, it & 2);
    switch (ri(0, 10)) {
      case 0: c.d_model = ri(-8, 300); break;
      case 1: c.n_heads = ri(-1, 9); break;
      case 2: c.max_nodes = ri(-2, 80); break;
      case 3: c.logit_hi = ri(-5, 600); break;
      case 4: c.feature_slots = ri(-2, 12); break;
      case 5: c.dtype = ri(-1, 3); break;
      case 6: c.n_prompts = ri(-1, 5); break;
      case 7: c.draft_input = ri(-1, 2); break;
      case 8: c.relax_k = ri(-1, 70); break;
      case 9: c.norm_mode = ri(-1, 2); break;
      default: break;
    }
    size_t a = 0, b = 0, d = 0;
    vvs_status st = vvs_query_sizes(&c, &a, &b, &d);
    if (st == VVS_OK && (a == 0 || b == 0 || d == 0)) { printf("empty buffer sizes accepted\n"); return 1; }
  }
  // 2b. tiles: every plan covers its columns exactly and stays inside a section; the residual projections change their tiles where
  // measurement put the line (rows of d 1280: more than 512 tiles of 64 x 64; at least 160 of 192 x 128)
  {
    vvs_config c = base_config(true, false);
    c.d_model = 1280; c.n_heads = 20; c.d_ff = 3456; c.n_prompts = 32;
    vvs::Ctx xl;
    std::string err;
    if (vvs::plan_sizes(&c, &xl, &err) != VVS_OK) { printf("XL plan: %s\n", err.c_str()); return 1; }
    for (int m = 1; m <= 6000; ++m) {
      const int want = m <= 352 ? 32 : m <= 1600 ? 64 : m <= 2880 ? 128 : 192;
      const vvs::GemmPlan r = vvs::plan_resid(&xl, m), q = vvs::plan_gemm(&xl, m, 3 * 1280, 1280, 1280), g = vvs::plan_gemm(&xl, m, 2 * 3456, 1280);
      if (r.bm != want || 1280 % r.bn || r.shared != (r.bm >= 128)) { printf("residual projection of %d rows: tiles of %d x %d\n", m, r.bm, r.bn); return 1; }
      // (more than two 64 x 64 workgroups per CU: no projection but the residual ones stays on tiles with operands of their own)
      const int rows64 = (m + 63) / 64;
      if (m > 192 && (q.shared != (rows64 * 60 > 512) || g.shared != (rows64 * 108 > 512))) { printf("%d rows: q/k/v or gate/up on the wrong side of 512 tiles\n", m); return 1; }
      if (1280 % q.bn || 6912 % g.bn) { printf("%d rows: a tile of %d or %d columns\n", m, q.bn, g.bn); return 1; }
    }
    // the partial-sum buffer holds every number of rows, not only the multiples of 32 it was planned at
    for (int wide = 0; wide < 2; ++wide) {
      vvs_config w = c;
      if (wide) { w.d_model = 4096; w.n_heads = 32; w.d_ff = 11008; w.max_nodes = 31; w.n_prompts = 6; }
      vvs::Ctx k;
      if (vvs::plan_sizes(&w, &k, &err) != VVS_OK) { printf("plan: %s\n", err.c_str()); return 1; }
      const int d = w.d_model, shapes[4][2] = {{3 * d, d}, {d, d}, {2 * w.d_ff, d}, {d, w.d_ff}};
      for (int m = 1; m <= k.Mmax; ++m)
        for (auto& sh : shapes) {
          const vvs::GemmPlan p = vvs::plan_gemm(&k, m, sh[0], sh[1]);
          if ((p.splits > 1 || sh[0] == d) && (size_t)p.splits * m * sh[0] > k.gemm_out_elems) { printf("%d rows: partial sums do not fit\n", m); return 1; }
        }
    }
    // ... and every projection of every shape, also where two have the same columns or the same contraction (d_ff of d / 2, 1.5 d, 2 d):
    // what forward_t launches with partial sums, each with the plan its launch takes
    long undersized = 0, checked = 0;
    for (int it = 0; it < 2000; ++it) {
      vvs_config w = base_config(true, it % 5 == 4);
      const int dh = ri(0, 1) ? 128 : 64, d = w.d_model = ri(1, 4096 / 128) * 128;
      w.n_layers = 1; w.n_heads = d / dh; w.max_nodes = ri(0, dh == 128 ? 31 : 63); w.n_prompts = ri(1, 8); w.grid_h = w.grid_w = ri(4, 24);
      w.prefix_len = ri(1, 120); w.norm_mode = it / 4 & 1;
      if (it % 8 == 6) { w.n_prompts = 1; w.grid_h = w.grid_w = 4; w.prefix_len = 1; }   // a verify call is the widest there is
      const int F = w.d_ff = it % 4 == 0 ? 2 * d : it % 4 == 1 ? d / 2 : it % 4 == 2 ? d / 2 * 3 : ri(std::max(1, d / 256), d / 64 * 3) * 64;
      vvs::Ctx k;
      if (vvs::plan_sizes(&w, &k, &err) != VVS_OK) { printf("plan: %s\n", err.c_str()); return 1; }
      if (vvs::plan_fused(&k, 1)) continue;                  // takes no partial sums
      auto sums = [&](int m, int n, int kk, int splits) {
        ++checked;
        if ((size_t)splits * m * n <= k.gemm_out_elems) return;
        if (++undersized <= 3) printf("d %d, d_ff %d, norm mode %d, %d rows: partial sums of %d columns over %d do not fit\n", d, F, w.norm_mode, m, n, kk);
      };
      auto need = [&](int m, int n, int kk) { sums(m, n, kk, vvs::plan_partial(&k, m, n, kk).splits); };
      for (int m32 = 32; m32 <= k.Mmax; m32 += 32)
        for (int m : {m32, m32 - ri(1, 31)}) {
          const vvs::GemmPlan q = vvs::plan_qkv(&k, m), gu = vvs::plan_gate_up(&k, m);
          if (q.splits > 1 && (m + q.bm - 1) / q.bm * (3 * d / q.bn) < 160) sums(m, 3 * d, d, q.splits);
          if (gu.splits > 1) sums(m, 2 * F, d, gu.splits);
          need(m, d, d);
          need(m, d, F);
          if (w.draft_input) need(m, d, 2 * d);
        }
    }
    if (undersized || checked < 300000) { printf("%ld of %ld launches overrun the partial sums\n", undersized, checked); return 1; }
    vvs::Ctx odd = xl;                                       // a third of 640 columns: 256-column tiles would cross it
    odd.d = 640;
    for (int m = 1; m <= 20000; m += 97)
      if (640 % vvs::plan_gemm(&odd, m, 3 * 640, 640, 640).bn) { printf("%d rows: a tile crosses the q / k / v thirds\n", m); return 1; }
  }
  // 2c. all layers in one launch: only where the device has a CU for each of its workgroups
  for (int cus : {256, 304, 255, 128, 32}) {
    vvs_config c = base_config(true, false);
    Dev mem;
    mem.alloc(c);
    vvs_ctx* ctx = nullptr;
    g_cus = cus;
    if (vvs_create(&c, mem.akv, mem.aws, mem.apw, &ctx) != VVS_OK) { printf("create with %d CUs: %s\n", cus, vvs_last_error(nullptr)); return 1; }
    for (int t = 1; t <= 70; ++t)
      if (vvs::layers_in_one_launch((const vvs::Ctx*)ctx, t) != (cus >= 256 && 6 * t <= 256)) { printf("%d CUs, %d tokens: one launch %d\n", cus, t, (int)(cus < 256)); return 1; }
    vvs_destroy(ctx);
  }
  g_cus = 256;
  // ... up to the rows where it stops paying: d, heads, d_ff, norm mode, the limit; each side of every line of few_rows and few_wide_rows
  for (const auto& s : {std::array<int, 5>{768, 12, 2048, 0, 224}, {768, 12, 7680, 0, 160}, {768, 12, 8192, 0, 128}, {768, 12, 9216, 0, 96}, {512, 8, 12288, 0, 64}, {512, 8, 2048, 0, 256},
                        {256, 4, 24576, 0, 32}, {192, 3, 512, 0, 256}, {1280, 20, 3456, 0, 192}, {768, 12, 7168, 1, 128}, {768, 12, 7680, 1, 64}, {960, 15, 9600, 0, 128}, {1024, 16, 8192, 0, 128},
                        {1024, 16, 10240, 0, 64}, {1088, 17, 11264, 0, 64}, {1792, 14, 23040, 0, 64}, {1792, 14, 25088, 0, 32}, {2048, 16, 5504, 0, 128}, {2048, 16, 8192, 0, 64},
                        {2560, 20, 12288, 0, 64}, {2560, 20, 12800, 0, 32}, {3520, 55, 13440, 0, 32}, {3584, 28, 12544, 0, 0}, {3584, 28, 12288, 0, 64}, {3840, 60, 12800, 0, 0}, {3840, 30, 1920, 0, 64}, {3840, 30, 1536, 0, 32},
                        {4096, 32, 2048, 0, 32}, {4096, 32, 11008, 0, 64}, {4096, 32, 12288, 0, 64}, {4096, 32, 14336, 0, 0}, {4160, 65, 4160, 0, 0}}) {
    vvs_config c = base_config(true, false);
    c.n_layers = 1; c.d_model = s[0]; c.n_heads = s[1]; c.d_ff = s[2]; c.norm_mode = s[3]; c.n_prompts = 4; c.max_nodes = 63; c.grid_h = c.grid_w = 16;
    if (s[0] / s[1] == 128) { c.n_prompts = 8; c.max_nodes = 31; }
    vvs::Ctx k;
    std::string err;
    if (vvs::plan_sizes(&c, &k, &err) != VVS_OK) { printf("plan: %s\n", err.c_str()); return 1; }
    k.cus = 256;
    vvs_config drafter = c;
    drafter.draft_input = 1;
    vvs::Ctx dr;
    if (vvs::plan_sizes(&drafter, &dr, &err) != VVS_OK) { printf("plan: %s\n", err.c_str()); return 1; }
    dr.cus = 256;                                              // wide drafters and narrow ones never, the others as targets
    if (vvs::layers_in_one_launch(&dr, 1) != (vvs::plan_fused(&k, 1) && s[0] / s[1] == 64 && s[0] >= 256)) { printf("drafter of d %d, d_ff %d\n", s[0], s[2]); return 1; }
    for (int t = 1; t <= k.Tmax; ++t)
      if (vvs::layers_in_one_launch(&k, t) != (k.R * t <= s[4])) { printf("d %d, d_ff %d, %d rows: one launch %d\n", s[0], s[2], k.R * t, (int)vvs::layers_in_one_launch(&k, t)); return 1; }
  }
  // 3. the call sequences, launchers replaced: target + drafter, fp32 and bf16 planning
  for (int bf16 = 0; bf16 < 2; ++bf16) {
    vvs_config tc = base_config(bf16, false), dc = base_config(bf16, true);
    Dev td, dd;
    td.alloc(tc); dd.alloc(dc);
    vvs_ctx *tg = nullptr, *dr = nullptr;
    if (vvs_create(&tc, td.akv, td.aws, td.apw, &tg) != VVS_OK || vvs_create(&dc, dd.akv, dd.aws, dd.apw, &dr) != VVS_OK) {
      printf("create failed: %s\n", vvs_last_error(nullptr)); return 1;
    }
    std::vector<const void*> wt(vvs_num_weight_tensors(&tc), (const void*)td.apw), wd(vvs_num_weight_tensors(&dc), (const void*)dd.apw);
    int32_t dummy_i[4096]; float dummy_f[64];
    memset(dummy_i, 0, sizeof(dummy_i));
    void* fake = dummy_i;    // pointers handed to launchers are never dereferenced by the stand-ins
    if (vvs_verify(tg, 0, nullptr, nullptr, nullptr, nullptr, dummy_f, VVS_STRICT, dummy_i, dummy_i, dummy_i, nullptr) != VVS_ESTATE) { printf("verify before prefill\n"); return 1; }
    if (vvs_load_weights(tg, wt.data(), (int)wt.size(), nullptr) != VVS_OK || vvs_load_weights(dr, wd.data(), (int)wd.size(), nullptr) != VVS_OK) { printf("load\n"); return 1; }
    if (vvs_load_weights(dr, wd.data(), (int)wd.size() - 1, nullptr) == VVS_OK) { printf("short weight list accepted\n"); return 1; }
    if (vvs_draft(dr, tg, 3, nullptr, nullptr, 1, dummy_i, 0, nullptr, dummy_i, dummy_f, nullptr) != VVS_ESTATE) { printf("draft before prefill\n"); return 1; }
    if (vvs_prefill(tg, fake, nullptr, 7, dummy_i, dummy_f, dummy_i, nullptr) != VVS_OK) { printf("prefill: %s\n", vvs_last_error(tg)); return 1; }
    if (vvs_prefill(dr, fake, nullptr, 0, nullptr, dummy_f, dummy_i, nullptr) == VVS_OK) { printf("prefill on a drafter accepted\n"); return 1; }
    int ok_verify = 0, ok_draft = 0;
    for (int it = 0; it < 1500; ++it) {
      const int n = ri(0, 45);
      std::vector<int32_t> parent;
      random_tree(n, parent, it % 5 != 0);
      int n_post = it % 4 == 0 ? ri(0, 6) : 0;
      if (n_post && n >= n_post) {                              // hang the tree below a chain of unverified tokens
        for (int j = 1; j <= n; ++j) parent[j - 1] = j <= n_post ? j - 1 : std::max(parent[j - 1], (int32_t)n_post);
      }
      vvs_status st = vvs_verify_post(tg, n, n_post, n ? parent.data() : nullptr, nullptr, dummy_i, dummy_f, dummy_f, VVS_STRICT, dummy_i, dummy_i, dummy_i, nullptr);
      if (st == VVS_OK) {
        ++ok_verify;
        if (vvs_verify(tg, 0, nullptr, nullptr, nullptr, nullptr, dummy_f, VVS_STRICT, dummy_i, dummy_i, dummy_i, nullptr) != VVS_ESTATE) { printf("second verify without commit\n"); return 1; }
        if (vvs_kv_commit(tg, nullptr) != VVS_OK) { printf("commit\n"); return 1; }
        if (vvs_kv_commit(tg, nullptr) != VVS_ESTATE) { printf("double commit accepted\n"); return 1; }
      } else if (n > tc.max_nodes && st != VVS_ESIZE) { printf("oversized verify: status %d\n", st); return 1; }
      const int k = ri(0, 6), nu = ri(-1, 9);
      st = vvs_draft(dr, tg, n, n ? parent.data() : nullptr, nullptr, k, dummy_i, nu, it & 1 ? dummy_i : nullptr, dummy_i, dummy_f, nullptr);
      if (st == VVS_OK) ++ok_draft;
      (void)vvs_path_similarity(tg, n, n ? parent.data() : nullptr, nullptr, dummy_i, 0.8f, ri(0, 3), dummy_f, nullptr);
    }
    if (ok_verify < 200 || ok_draft < 50) { printf("too few valid calls: %d verify, %d draft\n", ok_verify, ok_draft); return 1; }
    (void)vvs_read_features(tg, dummy_f, dummy_i, nullptr);
    (void)vvs_debug_logits(tg, nullptr, nullptr, nullptr, nullptr);
    (void)vvs_debug_logits(dr, nullptr, nullptr, nullptr, nullptr);
    vvs_destroy(tg);
    vvs_destroy(dr);
    printf("dtype %d: %d verify calls and %d drafting calls passed the host checks\n", bf16, ok_verify, ok_draft);
  }
  printf("host fuzz ok, %ld launches reached the stand-ins\n", vvs::g_launches);
  return 0;
}
