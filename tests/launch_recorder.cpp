// Launch recorder: the host side of the library linked against a HIP runtime that runs nothing.  Every kernel launch,
// event record and stream wait is printed as one JSON line, with the memory ranges that matter to the tests, so
// that launch decisions, stream order and buffer extents can be checked on a machine without a GPU.  Device
// pointers are made-up addresses; nothing here reads or writes through them.
//
// usage: launch_recorder <call> key=value ...      (see main)
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../include/mace.h"
#include "gemm.h"
#include "kernels.h"

// ---------------------------------------------------------------- the runtime
static std::map<const void *, std::string> g_kernels;
static std::map<const void *, int> g_streams, g_events;
static dim3 g_grid, g_block;
static hipStream_t g_stream;
static uintptr_t g_next = (uintptr_t)1 << 44;

static void *fake(size_t bytes) {
  void *p = (void *)g_next;
  g_next += (bytes + ((size_t)1 << 20)) & ~(((size_t)1 << 20) - 1);      // a gap behind every buffer
  return p;
}
static int id_of(std::map<const void *, int> &m, const void *p) {
  auto it = m.find(p);
  return it != m.end() ? it->second : m[p] = (int)m.size();
}
static int stream_id(hipStream_t s) { return id_of(g_streams, s); }      // 0 = the caller's (null) stream
static const char *g_sep;
static void range(const char *kind, const void *p, size_t bytes) {
  printf("%s[\"%s\", %llu, %llu]", g_sep, kind, (unsigned long long)(uintptr_t)p, (unsigned long long)bytes);
  g_sep = ", ";
}
static void read_parts(const Parts &s) {
  if (s.p && s.stride) range("parts_in", s.p, (size_t)s.n * s.stride * 4);
}
template <typename T>
static const T &arg(void **a, int i) { return *(const T *)a[i]; }

static void describe(const std::string &k, void **a) {
  auto is = [&](const char *n) { return k.find(n) != std::string::npos; };
  if (is("gemm_bf16_w4_kernel") || is("gemm_bf16_dl_kernel")) {
    const GemmParams &p = arg<GemmParams>(a, 0);
    for (int g = 0; g < p.n_mg; ++g)
      if (p.k_splits[g] > 1 || p.mg[g].c_split_stride)
        range("parts_out", p.mg[g].c, (size_t)(p.k_splits[g] > 1 ? p.k_splits[g] : 1) * p.mg[g].c_split_stride * 4);
  } else if (is("skinny_kernel")) {
    const SkinnyParams &p = arg<SkinnyParams>(a, 0);
    printf("%s[\"skinny\", %llu, %d, %d, %d], [\"shares\", %d, %d]", g_sep, (unsigned long long)(uintptr_t)p.a, p.M, p.N, p.K, p.share, p.rest);
    g_sep = ", ";
  } else if (is("sum_parts_kernel")) {
    for (int i = 0; i < 3; ++i) read_parts(arg<SumRange>(a, i).parts);
  } else if (is("scale_split_kernel") || is("extract_kernel") || is("rmsnorm_bwd_kernel")) {
    read_parts(arg<Parts>(a, 0));
  } else if (is("swiglu_bwd_kernel")) {
    if (!arg<const void *>(a, 0)) read_parts(arg<Parts>(a, 1));
  } else if (is("swiglu_fwd_kernel")) {
    for (int i = 0; i < 2; ++i) read_parts(arg<SwigluRows>(a, i).gu_in);
  } else if (is("rmsnorm_fwd_kernel")) {
    for (int i = 0; i < 2; ++i) read_parts(arg<NormRows>(a, i).parts);
  } else if (is("rope_split_kernel")) {
    for (int i = 0; i < 2; ++i) read_parts(arg<RopeRows>(a, i).qkv);
  }
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { g_kernels[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t s) { g_grid = g; g_block = b; g_stream = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) { *g = g_grid; *b = g_block; *m = 0; *s = g_stream; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t, hipStream_t s) {
  printf("{\"op\": \"launch\", \"kernel\": \"%s\", \"stream\": %d, \"grid\": [%u, %u, %u], \"block\": %u, \"ranges\": [", g_kernels[f].c_str(), stream_id(s), g.x, g.y, g.z, b.x);
  g_sep = "";
  describe(g_kernels[f], a);
  printf("]}\n");
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { printf("{\"op\": \"record\", \"event\": %d, \"stream\": %d}\n", id_of(g_events, e), stream_id(s)); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { printf("{\"op\": \"wait\", \"event\": %d, \"stream\": %d}\n", id_of(g_events, e), stream_id(s)); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)fake(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)fake(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = fake(n); return hipSuccess; }
hipError_t hipFree(void *) { return hipSuccess; }
static bool g_uploads;      // print the fp64 arrays that are copied to the device
hipError_t hipMemcpy(void *, const void *src, size_t n, hipMemcpyKind) {
  if (g_uploads)
    for (size_t i = 0; i < n / 8; ++i) printf("{\"op\": \"upload\", \"value\": %.17g}\n", ((const double *)src)[i]);
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = fake((size_t)4 << 20); return hipSuccess; }
}

// ---------------------------------------------------------------- the calls
static std::map<std::string, std::string> g_opt;
static long long num(const char *k, long long dflt) { return g_opt.count(k) ? atoll(g_opt[k].c_str()) : dflt; }
static std::vector<int> list(const char *k) {
  std::vector<int> v;
  if (!g_opt.count(k)) return v;
  for (const char *s = g_opt[k].c_str(); *s;) {
    char *e;
    v.push_back((int)strtol(s, &e, 10));
    s = *e == ',' ? e + 1 : e;
  }
  return v;
}
static void *buffer(const char *name, size_t bytes) {      // misalign=<name> moves one pointer by two bytes
  char *p = (char *)fake(bytes + 16);
  return g_opt.count("misalign") && g_opt["misalign"] == name ? p + 2 : p;
}
static int result(mace_handle_t h, int rc) {
  printf("{\"op\": \"return\", \"status\": %d, \"error\": \"%s\"}\n", rc, rc ? mace_last_error() : "");
  static mace_gemm_plan_t plan[256];
  int32_t n = 0;
  mace_launch_plan(h, plan, 256, &n);
  for (int i = 0; i < n; ++i)
    printf("{\"op\": \"plan\", \"name\": \"%s\", \"tile\": [%d, %d], \"k_splits\": %d, \"side\": %d, \"m\": %lld, \"n\": %lld, \"k\": %lld}\n",
           plan[i].name, plan[i].tile_m, plan[i].tile_n, plan[i].k_splits, plan[i].on_side_stream, (long long)plan[i].m, (long long)plan[i].n, (long long)plan[i].k);
  return 0;
}

// gemm_launch itself: groups=M,passes,slices[,M,passes,slices..] in the order given, N=, K=
static int raw_gemm() {
  const std::vector<int> v = list("groups");
  GemmParams p;
  memset(&p, 0, sizeof(p));
  p.K = (int)num("K", 4096);
  p.n_ns = 1;
  p.ns[0].N = (int)num("N", 4096);
  p.ns[0].b[0] = p.ns[0].b[1] = (const bf16_t *)fake(1);
  p.lda = p.ldb = p.K;
  p.ldc = p.ldr = p.ns[0].N;
  for (size_t i = 0; i + 2 < v.size(); i += 3) {
    GemmMGroup &g = p.mg[p.n_mg];
    g.a[0] = g.a[1] = (const bf16_t *)fake(1);
    g.M = v[i]; g.npass = v[i + 1];
    g.c_split_stride = (long long)g.M * p.ldc;
    g.c = fake((size_t)v[i + 2] * g.c_split_stride * 4);
    p.k_splits[p.n_mg++] = v[i + 2];
  }
  const char *why = nullptr;
  const hipError_t e = gemm_launch(0, 0, p, nullptr, &why);
  printf("{\"op\": \"return\", \"status\": %d, \"error\": \"%s\", \"groups\": [", (int)e, why ? why : "");
  for (int g = 0; g < p.n_mg; ++g) printf("%s[%d, %d, %d]", g ? ", " : "", p.mg[g].M, p.mg[g].npass, p.k_splits[g]);
  printf("]}\n");
  return 0;
}

// rope_sincos of every angle positions[i] * 1e4^(-2 j / 128), all digits
static int rope() {
  for (int pos : list("positions"))
    for (int j = 0; j < 64; ++j) {
      double s, c;
      rope_sincos((double)pos * std::pow(1e4, -2.0 * j / 128), s, c);
      printf("{\"op\": \"rope\", \"angle\": %.17g, \"sin\": %.17g, \"cos\": %.17g}\n", (double)pos * std::pow(1e4, -2.0 * j / 128), s, c);
    }
  return 0;
}

int main(int argc, char **argv) {
  const std::string call = argc > 1 ? argv[1] : "";
  for (int i = 2; i < argc; ++i) {
    const char *e = strchr(argv[i], '=');
    if (!e) return 2;
    g_opt[std::string(argv[i], e - argv[i])] = e + 1;
  }
  (void)stream_id(nullptr);
  if (call == "gemm") return raw_gemm();
  if (call == "rope") return rope();
  mace_model_t m = {(int32_t)num("d", 1024), (int32_t)num("hq", 8), (int32_t)num("hkv", 8), (int32_t)num("hd", 128), (int32_t)num("F", 2816), (int32_t)num("V", 4096),
                    1e-6f, g_opt.count("theta") ? (float)atof(g_opt["theta"].c_str()) : 1e4f, num("bf16", 1) ? MACE_BF16 : MACE_F32};
  mace_handle_t h;
  g_uploads = call == "create";
  if (mace_create(&h, &m) != MACE_OK) { fprintf(stderr, "%s\n", mace_last_error()); return 3; }
  if (g_uploads) return 0;
  if (num("single_stream", 0)) mace_set_option(h, MACE_OPT_SINGLE_STREAM, 1);

  if (call == "product") {      // mace_gemm_bf16: la= lb= M= N= K=, ldc= ldr= beside N, out_bf16= resid= swiglu= kernel=, two= a second term of A, keep= what the forward keeps
    mace_gemm_desc_t p;
    memset(&p, 0, sizeof(p));
    p.layout_a = (int32_t)num("la", 0); p.layout_b = (int32_t)num("lb", 0);
    p.M = (int32_t)num("M", 64); p.N = (int32_t)num("N", 64); p.K = (int32_t)num("K", 64);
    p.lda = p.layout_a ? p.M : p.K; p.ldb = p.layout_b ? p.N : p.K;
    p.ldc = num("ldc", p.N); p.ldr = num("ldr", p.ldc);
    p.a = fake(256); p.b = fake(256); p.c = fake(256);
    if (num("two", 0)) p.a_lo = fake(256);
    if (num("swiglu", 0) == 1) p.b_up = fake(256);
    if (num("keep", 0)) { p.c_lo = fake(256); p.c_gu = fake(256); }
    if (num("swiglu", 0) == 2) p.c_gu = fake(256);
    p.out_bf16 = (int32_t)num("out_bf16", 0); p.swiglu = (int32_t)num("swiglu", 0); p.kernel = (int32_t)num("kernel", 0);
    p.resid_kind = (int32_t)num("resid", 0);
    if (p.resid_kind) p.resid = fake(256);
    return result(h, mace_gemm_bf16(h, &p, nullptr));
  }
  if (call == "workspace") {      // decode=counts contexts=lengths: the bytes of every pair, tokens=, ft_tokens= other rows
    for (int n : list("decode"))
      for (int c : list("contexts")) {
        const int other = (int)num("tokens", 0), Tf = (int)num("ft_tokens", 0);
        printf("{\"op\": \"workspace\", \"decode\": %d, \"context\": %d, \"bytes\": %zu}\n", n, c, mace_workspace_bytes(h, n + other + Tf, Tf, n, c, 0));
      }
    return 0;
  }

  // batch: prefill=lengths decode=contexts ft=lengths
  const std::vector<int> pre = list("prefill"), ctx = list("decode"), ft = list("ft");
  std::vector<int32_t> seg{0}, lens(ctx.begin(), ctx.end());
  int Tf = 0, max_ctx = 0;
  for (int L : pre) seg.push_back(seg.back() + L);
  for (int c : ctx) { seg.push_back(seg.back() + 1); max_ctx = c > max_ctx ? c : max_ctx; }
  const int Ti = seg.back();
  for (int L : ft) { seg.push_back(seg.back() + L); Tf += L; }
  mace_batch_t b;
  memset(&b, 0, sizeof(b));
  b.n_prefill = (int)pre.size(); b.n_decode = (int)ctx.size(); b.n_ft_seq = (int)ft.size(); b.n_tokens = Ti + Tf;
  b.seg_offsets_host = seg.data();
  b.seg_offsets = (const int32_t *)fake(1 << 20); b.positions = (const int32_t *)fake(1 << 20);
  b.slot_mapping = (const int32_t *)fake(1 << 20);
  b.context_lens_host = lens.data(); b.context_lens = (const int32_t *)fake(1 << 20);
  b.block_tables = (const int32_t *)fake(1 << 20); b.max_blocks_per_req = max_ctx / 16 + 1;
  mace_kv_cache_t cache = {fake((size_t)1 << 30), fake((size_t)1 << 30), 1 << 20, 16};

  const size_t d = m.d_model, qd = (size_t)m.n_q_heads * m.head_dim, kd = (size_t)m.n_kv_heads * m.head_dim, F = m.d_ff, V = m.vocab, e = 4;
  mace_layer_w_t w = {buffer("g_attn", d * e), buffer("wq", qd * d * e), buffer("wk", kd * d * e), buffer("wv", kd * d * e), buffer("wo", qd * d * e),
                      buffer("g_mlp", d * e), buffer("w_gate", F * d * e), buffer("w_up", F * d * e), buffer("w_down", F * d * e)};
  mace_lora_t l = {buffer("a_q", 64 * d * e), buffer("b_q", 64 * qd * e), buffer("a_k", 64 * d * e), buffer("b_k", 64 * kd * e), buffer("a_v", 64 * d * e),
                   buffer("b_v", 64 * kd * e), buffer("a_o", 64 * qd * e), buffer("b_o", 64 * d * e), (int32_t)num("lora", 0), 2.0f};
  const size_t rows = (size_t)(Ti + Tf), work_bytes = (size_t)num("work", (long long)mace_workspace_bytes(h, Ti + Tf, Tf, b.n_decode, max_ctx, (int32_t)num("n", 0)));
  void *x = buffer("x", rows * d * e), *y = buffer("y", rows * d * 4), *saved = buffer("saved", mace_fwd_saved_bytes(h, Tf) + 256), *work = buffer("work", work_bytes);
  printf("{\"op\": \"work\", \"ptr\": %llu, \"bytes\": %llu}\n", (unsigned long long)(uintptr_t)work, (unsigned long long)work_bytes);
  const int acc = (int)num("accumulate", 0);
  if (call == "fwd")
    return result(h, l.rank ? mace_hybrid_layer_fwd_lora(h, &w, &l, &b, &cache, x, (float *)y, saved, work, work_bytes, nullptr)
                            : mace_hybrid_layer_fwd(h, &w, &b, &cache, x, (float *)y, saved, work, work_bytes, nullptr));
  if (call == "bwd") {
    float *dy = (float *)buffer("dy", (size_t)Tf * d * 4), *dx = (float *)buffer("dx", (size_t)Tf * d * 4);
    if (l.rank) {
      mace_lora_grads_t g = {(float *)buffer("", 64 * d * 4), (float *)buffer("", 64 * qd * 4), (float *)buffer("", 64 * d * 4), (float *)buffer("", 64 * kd * 4),
                             (float *)buffer("", 64 * d * 4), (float *)buffer("", 64 * kd * 4), (float *)buffer("", 64 * qd * 4), (float *)buffer("", 64 * d * 4)};
      return result(h, mace_hybrid_layer_bwd_lora(h, &w, &l, &b, x, dy, saved, dx, &g, acc, work, work_bytes, nullptr));
    }
    mace_layer_grads_t g = {(float *)buffer("", d * 4), (float *)buffer("", qd * d * 4), (float *)buffer("", kd * d * 4), (float *)buffer("", kd * d * 4), (float *)buffer("", qd * d * 4),
                            (float *)buffer("", d * 4), (float *)buffer("", F * d * 4), (float *)buffer("", F * d * 4), (float *)buffer("", F * d * 4)};
    return result(h, mace_hybrid_layer_bwd(h, &w, &b, x, dy, saved, dx, &g, acc, work, work_bytes, nullptr));
  }
  if (call == "logits") {
    const int n = (int)num("n", 1);
    return result(h, mace_next_token_logits(h, (const float *)y, (const int32_t *)fake(1 << 20), n, buffer("g_final", d * e), buffer("w_lm", V * d * e),
                                            (float *)fake((size_t)n * V * 4), nullptr, work, work_bytes, nullptr));
  }
  fprintf(stderr, "unknown call %s\n", call.c_str());
  return 2;
}
