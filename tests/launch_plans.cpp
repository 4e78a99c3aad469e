// Host-only sweep of the library's launches (test_launch_plans.py builds and runs it; no GPU).  The functions of
// the HIP runtime that launch something are defined here, in the program, and so take the place of the runtime's: a
// launch is looked at instead of run.  Device pointers are made-up addresses that nothing reads.
//
// Checked for every launch of gemm_tile with a split k range: its partial tiles, as the kernel that is launched
// lays them out, lie inside the part of the workspace that is theirs.
//
// With the argument "routes" it reads calls from its input, "entry n k m batch dtype trans_a trans_b" a line, and prints
// for each the result and the kernels launched; with "grids" each kernel's workgroups behind its name.
#include <cstdio>
#include <cstring>
#include <map>
#include <random>
#include <string>
#include <vector>
#include "gecc_internal.h"

using namespace gecc;

// (the library registers its kernels before this program's own objects are made)
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static struct { dim3 grid, block; size_t lds; hipStream_t st; } g_cfg;
static gecc_ctx* g_ctx;
static GemmSide g_side;      // of the last launch of gemm_tile
static long g_launches, g_scans, g_narrow_split, g_main_split, g_bad;
static std::string g_case;

static std::vector<std::string> g_names;      // kernels of the call, in order
static bool g_grids;

static void look_at(const std::string& name, void** args) {
  ++g_launches;
  g_names.push_back(g_grids ? name + ":" + std::to_string((long)g_cfg.grid.x * g_cfg.grid.y * g_cfg.grid.z) : name);
  if (name.find("rowdot") != std::string::npos || name.find("coldot") != std::string::npos) ++g_scans;
  if (name.find("gemm_tile") == std::string::npos) return;
  const GemmArgs& a = *static_cast<const GemmArgs*>(args[0]);
  // the scans beside the product: every one has a workgroup, before the product's or behind
  const GemmSide& s = g_side = *static_cast<const GemmSide*>(args[1]);
  const int64_t own = (s.own + 7) / 8 * 8, behind = (s.groups - s.lead) * 8;
  if (s.groups > 0 && (s.lead_blocks < s.pg_items || s.lead_blocks > s.blocks || s.lead * 8 < s.lead_blocks || s.lead_blocks + behind < s.blocks ||
                       s.lead * 8 + own + behind != (int64_t)g_cfg.grid.x)) {
    if (++g_bad <= 8) printf("BAD %s: %d workgroups of scans, %d before the product's, grid %u\n", g_case.c_str(), s.blocks, s.lead_blocks, g_cfg.grid.x);
  }
  if (a.ksplit <= 1) return;
  const int64_t tile = name.find("ELi128EEEv") != std::string::npos ? 128 : name.find("ELi64EEEv") != std::string::npos ? 64 : 0;
  const int64_t tiles = (a.n + tile - 1) / tile * ((a.m + tile - 1) / tile) * a.batch;
  const char* beg = reinterpret_cast<const char*>(a.split_part);
  const char* end = beg + tiles * a.ksplit * tile * tile * (int64_t)sizeof(float);
  // (blocked mode: the narrow products' partial tiles lie where the partial sums of the main one will be)
  const bool narrow = g_ctx->nbi > 0;
  ++(narrow ? g_narrow_split : g_main_split);
  const Layout& L = g_ctx->lay;
  const char* lo = g_ctx->ws + (narrow ? L.rowpart : L.ksplit);
  const char* hi = g_ctx->ws + (narrow ? L.synd : L.total);
  if (tile == 0 || tiles > SCAN_DONE_WORDS || beg < lo || end > hi) {
    if (++g_bad <= 8) printf("BAD %s: product %d x %d x %d, tile %d, ksplit %d: %lld bytes past the end of its room\n", g_case.c_str(), a.n, a.k, a.m,
                             (int)tile, a.ksplit, (long long)(end - hi));
  }
}

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device_name, unsigned, uint3*, uint3*, dim3*, dim3*, int*) {
  names()[host] = device_name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) { g_cfg = {grid, block, lds, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
  *grid = g_cfg.grid; *block = g_cfg.block; *lds = g_cfg.lds; *st = g_cfg.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) { look_at(names()[f], args); return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
}

// one encoded product; `off`: elements the operands start behind a 16-byte boundary
static int one(int n, int k, int m, int batch, int dtype, int ta, int tb, int bn, int bm, int pad, int off, const std::string& entry = "multiply") {
  gecc_params p{};
  p.n = n; p.k = k; p.m = m; p.batch = batch; p.dtype = dtype; p.trans_a = ta; p.trans_b = tb;
  p.lda = (ta ? n : k) + pad; p.ldb = (tb ? k : m) + pad; p.ldc = m + pad;
  p.stride_a = (int64_t)(ta ? k : n) * p.lda; p.stride_b = (int64_t)(tb ? m : k) * p.ldb; p.stride_c = (int64_t)n * p.ldc;
  p.weighted = 1; p.block_n = bn; p.block_m = bm;
  g_case = std::string(dtype == GECC_BF16 ? "bf16 " : "fp32 ") + std::to_string(n) + "x" + std::to_string(k) + "x" + std::to_string(m) + " batch " +
           std::to_string(batch) + " blocks " + std::to_string(bn) + "x" + std::to_string(bm) + " layout " + std::to_string(ta) + std::to_string(tb) +
           " pad " + std::to_string(pad) + " start " + std::to_string(off);
  g_names.clear();
  if (gecc_create(&g_ctx, &p) != GECC_OK) { ++g_bad; printf("BAD %s: refused\n", g_case.c_str()); return GECC_ERR_ARG; }
  const uintptr_t at = (uintptr_t)1 << 40, esz = dtype == GECC_BF16 ? 2 : 4;
  auto dev = [&](int i, uintptr_t bytes) { return reinterpret_cast<void*>(at * (i + 1) + bytes); };
  int rc = gecc_set_workspace(g_ctx, dev(0, 0), gecc_workspace_bytes(g_ctx));
  double *ap = static_cast<double*>(dev(3, 0)), *bp = static_cast<double*>(dev(4, 0)), *cp = static_cast<double*>(dev(5, 0));
  void *A = dev(1, off * esz), *B = dev(2, off * esz);
  float* C = static_cast<float*>(dev(6, 0));
  if (!rc && entry == "multiply") rc = gecc_multiply(g_ctx, A, ap, B, bp, C, cp, nullptr, 0, nullptr);
  if (!rc && entry == "plain") rc = gecc_plain_gemm(g_ctx, A, B, C, nullptr);
  if (!rc && entry == "encode_a") rc = gecc_encode_a(g_ctx, A, ap, nullptr);
  if (!rc && entry == "correct") rc = gecc_correct(g_ctx, A, ap, B, bp, C, cp, static_cast<gecc_report*>(dev(7, 0)), nullptr);
  if (!rc && entry == "protected") rc = gecc_protected_gemm(g_ctx, A, B, C, ap, bp, cp, static_cast<gecc_report*>(dev(7, 0)), nullptr);
  if (rc) { ++g_bad; printf("BAD %s: %s\n", g_case.c_str(), gecc_strerror(rc)); }
  gecc_destroy(g_ctx);
  return rc;
}

static int routes() {
  char entry[32];
  int n, k, m, batch, dtype, ta, tb;
  while (scanf("%31s %d %d %d %d %d %d %d", entry, &n, &k, &m, &batch, &dtype, &ta, &tb) == 8) {
    const int rc = one(n, k, m, batch, dtype, ta, tb, 0, 0, 0, 0, entry);
    printf("%d", rc);
    for (const std::string& x : g_names) printf(" %s", x.c_str());
    printf("\n");
  }
  return 0;
}

int main(int argc, char** argv) {
  g_grids = argc > 1 && std::string(argv[1]) == "grids";
  if (g_grids || (argc > 1 && std::string(argv[1]) == "routes")) return routes();
  // (the sizes of test_narrow_products_of_blocked_mode_with_a_split_k_range first)
  one(4096, 264, 4096, 1, GECC_BF16, 0, 0, 2048, 2048, 0, 0);       // k no multiple of 64
  one(4096, 256, 4096, 1, GECC_BF16, 0, 0, 4096, 4096, 0, 0);       // a narrow product below 256 x 256 symbols
  one(2048, 384, 4096, 1, GECC_BF16, 0, 0, 1024, 1024, 0, 0);
  one(4096, 256, 4096, 1, GECC_BF16, 1, 1, 1024, 1024, 0, 1);       // operands that start off a 16-byte boundary
  one(4096, 512, 4096, 1, GECC_F32, 0, 1, 2048, 2048, 0, 0);
  if (g_narrow_split != 9) { ++g_bad; printf("BAD: %ld narrow products have a split k range, 9 should\n", g_narrow_split); }
  one(4096, 300, 4096, 1, GECC_BF16, 0, 0, 1024, 1024, 0, 0);
  one(8192, 300, 6144, 1, GECC_BF16, 0, 0, 8192, 6144, 0, 0);
  // the scans of the parity blocks: in the product's launch where that pays, else launches of their own
  auto scans = [](int n, int k, int m, int batch, int dtype, int ta, int tb) {
    const long before = g_scans;
    one(n, k, m, batch, dtype, ta, tb, 0, 0, 0, 0);
    return g_scans - before;
  };
  auto expect = [](bool ok, const char* what) { if (!ok) { ++g_bad; printf("BAD: scans of %s\n", what); } };
  expect(scans(128, 128, 128, 1, GECC_F32, 0, 0) == 0, "128^3");
  expect(scans(1024, 1024, 1024, 1, GECC_F32, 0, 0) == 0, "1024^3");
  expect(scans(1500, 1501, 1500, 1, GECC_BF16, 0, 1) == 0, "bf16 1500 x 1501 x 1500");
  expect(scans(600, 600, 600, 8, GECC_F32, 0, 1) > 0, "8 x 600^3 NT");
  expect(scans(2048, 2048, 2048, 1, GECC_F32, 0, 0) > 0, "2048^3");
  expect(scans(503, 301, 94, 307, GECC_BF16, 0, 0) > 0, "bf16 307 x 503 x 301 x 94");
  // before the product's workgroups where all run at once, else behind; column scans before row scans
  auto first = [&](int n, int k, int m, int ta, int tb, int dtype) { one(n, k, m, 1, dtype, ta, tb, 0, 0, 0, 0); return g_side.lead_blocks == g_side.blocks; };
  expect(first(1024, 1024, 1024, 0, 0, GECC_F32), "1024^3, all at once");
  expect(!first(1991, 1907, 220, 0, 0, GECC_F32) && g_side.lead_blocks == 1, "1991 x 1907 x 220, behind");
  expect(!first(2432, 3584, 256, 0, 0, GECC_BF16) && g_side.lead_blocks == 1, "bf16 2432 x 3584 x 256, behind");
  expect(!first(1632, 624, 2328, 1, 1, GECC_BF16) && g_side.j[0].kind == SIDE_COL && g_side.j[1].kind == SIDE_ROW, "bf16 1632 x 624 x 2328 TT, columns before rows");
  std::mt19937 rng(7);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (uint32_t)(hi - lo + 1)); };
  const int pads[] = {0, 0, 3, 8};
  for (int t = 0; t < 20000; ++t) {
    const int bn = 128 << pick(0, 5), bm = 128 << pick(0, 5), k = t % 3 ? pick(1, 1100) : 64 * pick(1, 64);
    one(bn * pick(1, 1 + 8192 / bn), k, bm * pick(1, 1 + 8192 / bm), 1, pick(0, 3) ? GECC_BF16 : GECC_F32, pick(0, 1), pick(0, 1), bn, bm, pads[pick(0, 3)], pick(0, 1));
  }
  for (int t = 0; t < 5000; ++t) {
    const int s = 1 << pick(0, 5);
    one(pick(1, 160) * s, pick(1, 160) * s, pick(1, 160) * s, pick(0, 3) ? 1 : pick(2, 64), pick(0, 1) ? GECC_BF16 : GECC_F32, pick(0, 1), pick(0, 1), 0, 0,
        pads[pick(0, 3)], pick(0, 1));
  }
  printf("%ld launches, k ranges: %ld narrow and %ld main products, bad: %ld\n", g_launches, g_narrow_split, g_main_split, g_bad);
  return g_bad || g_narrow_split < 1000 || g_main_split < 1000;
}
