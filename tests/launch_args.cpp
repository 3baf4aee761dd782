// What the launchers hand to the kernels, checked without a GPU: hipLaunchKernel is
// replaced by a recorder.  Linked against the library's objects by
// test_cpu_launch_args.py; each check is named on the command line and exits 0.
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "common.h"
#include "kernels/sample.h"

using namespace sq;

// The replaced launch looks for one pointer in the first bytes of the kernel's first
// argument (a struct larger than that).
static const void* g_wanted = nullptr;
static int g_launches = 0, g_found = 0;
static dim3 g_grid;                    // of the last launch
static const void* g_kernel = nullptr;

extern "C" hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void** args, size_t, hipStream_t) {
  g_kernel = kernel;
  ++g_launches;
  for (size_t o = 0; o + sizeof(void*) <= 96; o += sizeof(void*))
    if (g_wanted && memcmp((const char*)args[0] + o, &g_wanted, sizeof(void*)) == 0) ++g_found;
  return hipSuccess;
}
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3, size_t, hipStream_t) {
  g_grid = grid;
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* st) {
  *g = *b = dim3(1);
  *n = 0;
  *st = nullptr;
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

// whether the optimiser's kernel is handed the target of an average that starts at `begin` of 8
static bool ema_handed(long long begin) {
  static float p[8], g[8], m[8], v[8], target[1];
  int step = 0;
  sq_hparams hp{};
  g_wanted = target;
  g_launches = g_found = 0;
  const int s = adam(p, g, m, v, 8, &hp, &step, target, begin, nullptr, nullptr, nullptr);
  printf("status %d, %d launches, pointer handed %d times\n", s, g_launches, g_found);
  return s == SQ_OK && g_launches == 1 && g_found == 1;
}

// the few-row product that normalises its own input: 4 rows of H, weights [N, H]
struct LnCall {
  int n = 4, H = 256, A = 6;
  long long lk = 1;
  // launched (true) or refused without a launch
  bool launches(bool head) const {
    g_wanted = nullptr;
    g_launches = 0;
    const LnIn x{pre(), H, pre(), pre(), H, 1, nullptr, 0, 0};
    const MatArg W{weights(), H, lk, 0};
    float* out = pre();
    const int s = head ? gemm_ln_tanh_gauss(0, n, A, x, W, nullptr, nullptr, -5.f, 2.f, out, nullptr, nullptr, out, nullptr)
                       : gemm_ln(0, n, 2 * A, x, W, OutArg{out, 2 * A, 0, nullptr, 0, 0, 0}, nullptr);
    if (s != (g_launches ? SQ_OK : SQ_EINVAL) || g_launches > 1) printf("status %d, %d launches\n", s, g_launches);
    return s == SQ_OK && g_launches == 1;
  }
  static float* pre() { static float b[64 * 512] __attribute__((aligned(16))); return b; }
  static float* weights() { static float b[64 * 512] __attribute__((aligned(16))); return b; }
};

static bool ln_dropped(const float* buffer) {
  int owner = 0;
  fp32_drop_register(&owner, buffer, 64 * 512);
  const bool refused = !LnCall().launches(false) && !LnCall().launches(true);
  twin_unregister(&owner);
  return refused && LnCall().launches(false) && LnCall().launches(true);
}

static bool ln_form_refused(LnCall c) { return !c.launches(false) && !c.launches(true); }

// the tile (64 or 32) that a product of 2 x 64 t x 512 x 512 runs on: 16 t tiles of 64 x 64
static int tile(int bf16, int t, bool a_rows, bool b_rows) {
  float* p = LnCall::pre();   // not read
  const int M = 64 * t, N = 512, K = 512;
  const MatArg A{p, a_rows ? K : 1, a_rows ? 1 : M, (long long)M * K};
  const MatArg B{p, b_rows ? K : 1, b_rows ? 1 : N, (long long)N * K};
  g_launches = 0;
  const int s = gemm(bf16, M, N, K, 2, A, B, OutArg{p, N, (long long)M * N, nullptr, 0, 0, 0}, nullptr, 0, nullptr);
  if (s != SQ_OK || g_launches != 1 || (int)g_grid.z != 2) return 0;
  return M / (int)g_grid.x;
}

static bool tile_lines() {
  // {bfloat16, A's and B's rows k-contiguous, t, tile} on both sides of every line
  const int want[][5] = {{0, 1, 1, 15, 32}, {0, 1, 1, 16, 64}, {0, 1, 1, 17, 32}, {0, 1, 1, 21, 32}, {0, 1, 1, 22, 64},
                         {0, 1, 0, 16, 64}, {0, 1, 0, 17, 32}, {0, 1, 0, 25, 32}, {0, 1, 0, 26, 64},
                         {0, 0, 0, 16, 64}, {0, 0, 0, 17, 32}, {0, 0, 0, 25, 32}, {0, 0, 0, 26, 64},
                         {1, 1, 1, 16, 32}, {1, 1, 1, 27, 32}, {1, 1, 1, 28, 64}, {1, 0, 0, 27, 32}, {1, 0, 0, 28, 64}};
  bool ok = true;
  for (const auto& w : want) {
    const int got = tile(w[0], w[3], w[1], w[2]);
    if (got != w[4]) printf("bf16 %d rows %d %d, %d tiles: %d\n", w[0], w[1], w[2], 16 * w[3], got);
    ok = ok && got == w[4];
  }
  return ok;
}

// the kernel that a product of Z x 512 x 512 x K runs on (256 Z workgroups of the 32 x 32 tile)
static const void* kernel(int bf16, int Z, int K, bool strided) {
  float* p = LnCall::pre();   // not read
  const int N = 512, ld = (K + 3) / 4 * 4;
  const MatArg A{p, strided ? 1 : ld, strided ? N : 1, (long long)ld * N};
  g_launches = 0;
  const int s = gemm(bf16, N, N, K, Z, A, A, OutArg{p, N, (long long)N * N, nullptr, 0, 0, 0}, nullptr, 0, nullptr);
  return s == SQ_OK && g_launches == 1 && g_grid.x == 16 ? g_kernel : nullptr;
}

static bool register_groups() {
  // {bfloat16, strided, Z, K, Z, K, one kernel} across the lines between groups of one and two chunks
  const int want[][7] = {{0, 0, 1, 2048, 1, 2049, 0}, {1, 0, 1, 2048, 1, 2049, 0}, {0, 1, 1, 64, 1, 4096, 1},
                         {0, 1, 2, 1024, 2, 1025, 0}, {1, 1, 2, 2048, 2, 2049, 0}, {0, 0, 2, 64, 2, 4096, 1},
                         {0, 1, 3, 2047, 3, 2048, 0}, {1, 1, 3, 4095, 3, 4096, 0}, {1, 0, 3, 64, 3, 4096, 1},
                         {0, 1, 4, 255, 4, 256, 0},   {0, 1, 5, 511, 5, 512, 0},   {0, 0, 5, 511, 5, 512, 1},
                         {0, 1, 1, 512, 2, 512, 1},   {0, 1, 2, 512, 3, 512, 0}};
  bool ok = true;
  for (const auto& w : want) {
    const void* a = kernel(w[0], w[2], w[3], w[1]);
    const void* b = kernel(w[0], w[4], w[5], w[1]);
    const bool good = a && b && (a == b) == (w[6] != 0);
    if (!good) printf("bf16 %d strided %d: %d x K %d and %d x K %d\n", w[0], w[1], w[2], w[3], w[4], w[5]);
    ok = ok && good;
  }
  return ok;
}

// whether the encoder's launch reads frames `off` bytes off their alignment (k = 4: raw, k = 1: a ring's)
static bool frames_read(int k, int off) {
  const uint8_t* f = (const uint8_t*)LnCall::pre() + off;   // not read
  const float* b[3] = {};
  float* h[3] = {};
  SampleArgs sa{};
  sa.B = 2;
  g_launches = 0;
  const int s = encoder_fused_fwd_squint(sa, f, f, 16 * k, 16 * k, 9, 32, 3, k, nullptr, nullptr, b, h, nullptr, nullptr);
  return s == SQ_OK && g_launches == 1;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "adam_average")) return ema_handed(0) && ema_handed(7) ? 0 : 1;
  if (!strcmp(what, "adam_empty_average")) return !ema_handed(8) ? 0 : 1;
  if (!strcmp(what, "ln_dropped_weights")) return ln_dropped(LnCall::weights()) ? 0 : 1;
  if (!strcmp(what, "ln_dropped_input")) return ln_dropped(LnCall::pre()) ? 0 : 1;
  if (!strcmp(what, "ln_forms")) {
    LnCall rows, width, strided, wide;
    rows.n = 17;
    width.H = 320;
    strided.lk = 2;
    wide.A = 17;   // more head columns than one tile
    return ln_form_refused(rows) && ln_form_refused(width) && ln_form_refused(strided) && !wide.launches(true) ? 0 : 1;
  }
  if (!strcmp(what, "tile_lines")) return tile_lines() ? 0 : 1;
  if (!strcmp(what, "register_groups")) return register_groups() ? 0 : 1;
  if (!strcmp(what, "frame_alignment")) {
    const int want[][3] = {{4, 0, 1}, {4, 4, 1}, {4, 12, 1}, {4, 2, 0}, {1, 0, 1}, {1, 1, 1}, {1, 6, 1}};
    bool ok = true;
    for (const auto& w : want) {
      const bool read = frames_read(w[0], w[1]);
      if (read != (w[2] != 0)) printf("k = %d, %d bytes off: %d\n", w[0], w[1], read);
      ok = ok && read == (w[2] != 0);
    }
    return ok ? 0 : 1;
  }
  printf("unknown check '%s'\n", what);
  return 2;
}
