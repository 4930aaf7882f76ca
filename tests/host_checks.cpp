// Host-only checks of the WINO library's C ABI, built with AddressSanitizer
// and UndefinedBehaviorSanitizer on the host code (tests/test_abi_cpu.py
// builds and runs it): every path here returns before any HIP call, so it
// runs without a GPU.  Exits non-zero on the first failed check.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include <vector>

#include "kernels.h"
#include "wino.h"

static int g_checks = 0;
#define CHECK(cond)                                                        \
  do {                                                                     \
    ++g_checks;                                                            \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond); \
      std::exit(1);                                                        \
    }                                                                      \
  } while (0)

static wino_model_config tiny_cfg() {
  wino_model_config c{};
  c.n_layers = 2; c.d_model = 256; c.n_heads = 4; c.head_dim = 64; c.d_ff = 704; c.vocab = 4096;
  c.rope_theta = 10000.f; c.rms_eps = 1e-5f;
  return c;
}

static wino_params params(int B, int P, int G, int Lb, int mask, float t1 = 0.7f, float t2 = 0.9f) {
  wino_params p{};
  p.batch = B; p.prompt_len = P; p.gen_len = G; p.block_len = Lb; p.mask_id = mask;
  p.tau1 = t1; p.tau2 = t2;
  return p;
}

// End of n_main workgroups of length T and n_units of length U dealt in turn to 32
// shader engines of 8 CUs, each taking its own in order on the slot that frees first.
static double simulated_makespan(long n_main, double T, long n_units, double U, int occ) {
  std::vector<std::vector<double>> free_at(32, std::vector<double>(8 * occ, 0.0));
  double end = 0;
  for (long i = 0; i < n_main + n_units; ++i) {
    std::vector<double>& f = free_at[i % 32];
    size_t first = 0;
    for (size_t j = 1; j < f.size(); ++j) if (f[j] < f[first]) first = j;
    f[first] += i < n_main ? T : U;
    end = std::max(end, f[first]);
  }
  return end;
}

int main() {
  // the planners' dispatch model, around whole rounds of every occupancy
  for (int occ = 1; occ <= 3; ++occ)
    for (long round = 0; round <= 2; ++round)
      for (long d : {-40L, -17L, -16L, -4L, 0L, 1L, 12L, 33L, 100L})
        for (long units : {0L, 1L, 6L, 30L, 31L, 32L, 96L, 520L})
          for (double U : {0.37, 0.62, 1.0}) {
            const long n = 256L * occ * round + d;
            if (n < 0) continue;
            const double want = simulated_makespan(n, 1.0, units, U, occ);
            CHECK(std::fabs(wino::dispatch_makespan(n, 1.0, units, U, occ) - want) < 1e-6);
          }

  // a GEMM's plan is worked out once: calls of shapes seen before (a step has about
  // ten) take a fraction of the first ones' time and give the same plan
  for (const bool residual : {false, true}) {
    double first = 0, later = 1;
    for (int K = 2560; K < 2560 + 4 * 64; K += 64) {  // (four sets of new shapes)
      std::vector<wino::GemmCall> calls;
      for (int m : {37, 544, 1444, 8704}) {
        wino::GemmCall c{};
        c.M = m; c.K = K;
        c.epi = wino::EPI_QKV_ROPE; c.N = 3 * 2560; c.rope.H = 20; c.rope.hd = 128;
        if (!residual) calls.push_back(c);
        c.rope.H = 40; c.rope.hd = 64;
        if (!residual) calls.push_back(c);
        c.epi = wino::EPI_SWIGLU; c.N = 2 * 7616; c.F = 7616;
        if (!residual) calls.push_back(c);
        c.epi = wino::EPI_RESIDUAL; c.N = 2560;
        if (residual) calls.push_back(c);
      }
      std::vector<int> plan, again;
      auto pass = [&](std::vector<int>& out) {
        out.clear();
        const auto t0 = std::chrono::steady_clock::now();
        for (wino::GemmCall c : calls) {
          if (residual) wino::plan_residual_gemm(c, (size_t)8 * 1024 * c.N);
          else c.tile = wino::gemm_tile_n(c);
          for (int v : {c.tile, c.splits, c.split_row0}) out.push_back(v);
        }
        return std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
      };
      first += pass(plan) / 4;
      for (int i = 0; i < 5; ++i) {
        later = std::min(later, pass(again));
        CHECK(plan == again);
      }
    }
    std::printf("plans: first %.1f us, later %.1f us\n", first * 1e6, later * 1e6);
    CHECK(later < first / 3);
  }

  // sizes
  wino_model_config cfg = tiny_cfg();
  const size_t w1 = wino_workspace_bytes(&cfg, 1, 112), w2 = wino_workspace_bytes(&cfg, 2, 112);
  CHECK(w1 > 0 && w2 > w1);
  CHECK(wino_workspace_bytes(nullptr, 1, 112) == 0 && wino_workspace_bytes(&cfg, 0, 112) == 0);
  wino_model_config big = cfg;
  big.n_layers = 32; big.d_model = 4096; big.n_heads = 32; big.head_dim = 128; big.d_ff = 12288;
  big.vocab = 126464;
  CHECK(wino_workspace_bytes(&big, 16, 544) > wino_workspace_bytes(&big, 1, 544));
  CHECK(wino_epilogue_workspace_bytes(8, 32, 126464) >= (size_t)8 * 32 * 8 * 20);
  CHECK(wino_epilogue_workspace_bytes(0, 32, 126464) == 0);

  // wino_create: arguments rejected before any device work
  wino_ctx* ctx = nullptr;
  wino_weights w{};
  CHECK(wino_create(nullptr, &w, 1, 112, &ctx) == WINO_ERR_INVALID_ARG);
  CHECK(wino_create(&cfg, &w, 0, 112, &ctx) == WINO_ERR_SHAPE);
  CHECK(std::strcmp(wino_last_error(nullptr), "max_batch or max_seq") == 0);
  wino_model_config bad = cfg;
  bad.head_dim = 96; bad.d_model = 384;
  CHECK(wino_create(&bad, &w, 1, 112, &ctx) == WINO_ERR_UNSUPPORTED);
  bad = cfg; bad.vocab = 4000;
  CHECK(wino_create(&bad, &w, 1, 112, &ctx) == WINO_ERR_UNSUPPORTED);
  bad = cfg; bad.rms_eps = NAN;
  CHECK(wino_create(&bad, &w, 1, 112, &ctx) == WINO_ERR_UNSUPPORTED);
  bad = cfg; bad.act_precision = 2;
  CHECK(wino_create(&bad, &w, 1, 112, &ctx) == WINO_ERR_UNSUPPORTED);
  CHECK(wino_create(&cfg, &w, 1, 112, &ctx) == WINO_ERR_INVALID_ARG);  // null weights
  CHECK(ctx == nullptr);

  // the workspace limit, with placeholder (never dereferenced) weight pointers
  std::vector<const void*> layer(cfg.n_layers, reinterpret_cast<const void*>(0x1000));
  const void* ph = reinterpret_cast<const void*>(0x1000);
  wino_weights fake{ph, layer.data(), layer.data(), layer.data(), layer.data(), layer.data(), layer.data(),
                    ph, ph, nullptr};
  char lim[64];
  std::snprintf(lim, sizeof lim, "%zu", w2 - 1);
  setenv("WINO_WORKSPACE_LIMIT", lim, 1);
  CHECK(wino_create(&cfg, &fake, 2, 112, &ctx) == WINO_ERR_NO_MEMORY && ctx == nullptr);
  setenv("WINO_WORKSPACE_LIMIT", "0", 1);
  CHECK(wino_create(&cfg, &fake, 1, 112, &ctx) == WINO_ERR_NO_MEMORY && ctx == nullptr);
  unsetenv("WINO_WORKSPACE_LIMIT");

  // entry points without a context
  wino_params p = params(1, 32, 64, 16, 4095);
  CHECK(wino_step(nullptr, &p, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr) ==
        WINO_ERR_INVALID_ARG);
  CHECK(wino_decode(nullptr, &p, nullptr, nullptr, nullptr, nullptr, 0, nullptr, nullptr, nullptr) ==
        WINO_ERR_INVALID_ARG);
  CHECK(wino_decode_block(nullptr, &p, nullptr, nullptr, nullptr, nullptr, nullptr) == WINO_ERR_INVALID_ARG);
  CHECK(wino_row_losses(nullptr, &p, nullptr, nullptr, nullptr, nullptr) == WINO_ERR_INVALID_ARG);
  CHECK(wino_debug_logits(nullptr, &p, nullptr, nullptr, nullptr, nullptr) == WINO_ERR_INVALID_ARG);
  CHECK(wino_debug_forward(nullptr, &p, nullptr, nullptr, 0, nullptr, nullptr) == WINO_ERR_INVALID_ARG);
  CHECK(wino_destroy(nullptr) == WINO_ERR_INVALID_ARG);
  CHECK(wino_profile(nullptr, 1) == WINO_ERR_INVALID_ARG);
  CHECK(wino_profile_read(nullptr, nullptr, nullptr, nullptr, nullptr) == WINO_ERR_INVALID_ARG);

  // standalone epilogue: host-side validation (placeholder device pointers)
  void* d = reinterpret_cast<void*>(0x1000);
  int32_t* di = reinterpret_cast<int32_t*>(0x1000);
  uint8_t* du = reinterpret_cast<uint8_t*>(0x1000);
  wino_params e = params(1, 0, 16, 16, 4095, NAN, 0.9f);
  CHECK(wino_epilogue(&e, 4096, d, di, du, nullptr, nullptr, d, 1 << 20, nullptr) == WINO_ERR_INVALID_ARG);
  e = params(1, 0, 16, 16, 5000);
  CHECK(wino_epilogue(&e, 4096, d, di, du, nullptr, nullptr, d, 1 << 20, nullptr) == WINO_ERR_INVALID_ARG);
  e = params(1, 0, 16, 16, 4095);
  CHECK(wino_epilogue(&e, 4100, d, di, du, nullptr, nullptr, d, 1 << 20, nullptr) == WINO_ERR_SHAPE);
  CHECK(wino_epilogue(&e, 4096, d, di, du, nullptr, nullptr, d, 16, nullptr) == WINO_ERR_SHAPE);
  CHECK(wino_epilogue(&e, 4096, nullptr, di, du, nullptr, nullptr, d, 1 << 20, nullptr) == WINO_ERR_INVALID_ARG);
  CHECK(wino_epilogue(&e, 4096, d, di, du, nullptr, nullptr, nullptr, 1 << 20, nullptr) == WINO_ERR_INVALID_ARG);
  e.tokens_per_step = -1;
  CHECK(wino_epilogue_noalloc(&e, 4096, d, di, du, nullptr, nullptr, nullptr) == WINO_ERR_INVALID_ARG);
  e = params(128, 0, 128, 128, 126463);
  CHECK(wino_epilogue_workspace_bytes(128, 128, 126464) > WINO_EPILOGUE_NOALLOC_MAX_BYTES);
  CHECK(wino_epilogue_noalloc(&e, 126464, d, di, du, nullptr, nullptr, nullptr) == WINO_ERR_SHAPE);

  // GEMM test entry point: the tile planner rejects shapes without a kernel
  CHECK(wino_debug_gemm(nullptr, d, 64, 128, 64, nullptr, nullptr) == WINO_ERR_INVALID_ARG);
  CHECK(wino_debug_gemm(d, d, 0, 128, 64, reinterpret_cast<float*>(d), nullptr) == WINO_ERR_SHAPE);
  CHECK(wino_debug_gemm(d, d, 64, 128, 40, reinterpret_cast<float*>(d), nullptr) == WINO_ERR_UNSUPPORTED);
  CHECK(wino_debug_gemm(d, d, 64, 100, 64, reinterpret_cast<float*>(d), nullptr) == WINO_ERR_UNSUPPORTED);

  // strings
  for (int s = -7; s <= 0; ++s) CHECK(wino_status_string(static_cast<wino_status>(s)) != nullptr);
  CHECK(wino_kernel_class_name(-1)[0] == 0 && wino_kernel_class_name(WINO_N_KERNEL_CLASSES)[0] == 0);
  for (int k = 0; k < WINO_N_KERNEL_CLASSES; ++k) CHECK(wino_kernel_class_name(k)[0] != 0);
  // the last failed wino_create on this thread (the workspace-limit case above)
  CHECK(std::strcmp(wino_last_error(nullptr), "workspace larger than WINO_WORKSPACE_LIMIT") == 0);

  std::printf("host checks ok: %d\n", g_checks);
  return 0;
}
