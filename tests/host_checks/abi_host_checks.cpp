// Host-side paths of the C-ABI under AddressSanitizer and UndefinedBehaviorSanitizer: argument validation, the
// workspace layout, context creation and destruction, calls out of order, the table look-ups.  Nothing here launches
// a kernel: every call either fails its checks on the host, only builds host state or ends in the stand-ins for the
// runtime's launch below, which note the launch's size, so the program runs with or without a GPU.  Built and run by tests/test_host_sanitizers.py; exit status 0 = every call answered as
// expected and no sanitizer report.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "adore_internal.h"

// In place of the runtime's, which want a device: what the top-K attention would launch.
static std::vector<dim3> launched_grid, launched_block;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  launched_grid.push_back(grid);
  launched_block.push_back(block);
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *, hipStream_t *) {
  *grid = launched_grid.back();
  *block = launched_block.back();
  return hipSuccess;
}
static int launches = 0, failing_launch = -1;   // the one that is refused, counted from 1
// A controller's input projection whose contraction is cut into slices is the one kernel with a grid in three dimensions:
// (W, x, gi, D, 3d', tokens, ...), a slice behind the other in gi.
struct SlicedProjection {
  const float *gi;
  int width, tokens, slices;
};
static std::vector<SlicedProjection> sliced;
extern "C" hipError_t hipLaunchKernel(const void *, dim3 grid, dim3, void **args, size_t, hipStream_t) {
  ++launches;
  if (grid.z > 1)
    sliced.push_back({*static_cast<float **>(args[2]), *static_cast<int *>(args[4]), *static_cast<int *>(args[5]), int(grid.z)});
  return hipSuccess;
}
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return launches == failing_launch ? hipErrorLaunchFailure : hipSuccess; }

static int failures = 0;
#define EXPECT(cond)                                                          \
  do {                                                                        \
    if (!(cond)) {                                                            \
      std::fprintf(stderr, "line %d: %s\n", __LINE__, #cond);                 \
      ++failures;                                                             \
    }                                                                         \
  } while (0)

static adore_config tiny() {
  adore_config c;
  std::memset(&c, 0, sizeof c);
  c.layers = 1; c.batch = 1; c.heads = 4; c.head_dim = 64; c.hidden = 256; c.cache_slots = 64; c.rebuild_budget = 8;
  c.max_positions = 384; c.ctrl_hidden = 64; c.dtype = ADORE_F32; c.pos_scale = 1.0f / 384; c.score_mode = ADORE_SCORE_STATIC;
  c.rope_base = 0.f;
  return c;
}

int main() {
  EXPECT(adore_abi_version() == ADORE_ABI_VERSION);
  // a pointer that is never dereferenced on the host: the library only stores it
  std::vector<unsigned char> backing(4096);
  void *fake = reinterpret_cast<void *>((reinterpret_cast<uintptr_t>(backing.data()) + 255) / 256 * 256);
  float *ffake = static_cast<float *>(fake);
  adore_weights wt;
  {
    void **p = reinterpret_cast<void **>(&wt);
    for (size_t i = 0; i < sizeof wt / sizeof(void *); ++i) p[i] = fake;
  }
  adore_config c = tiny();
  const size_t n = adore_workspace_bytes(&c);
  EXPECT(n > 0 && n % 256 == 0);
  EXPECT(adore_workspace_bytes(nullptr) == 0);
  adore_ctx *h = nullptr;
  EXPECT(adore_create(nullptr, &wt, fake, n, nullptr, &h) == ADORE_E_INVALID);
  EXPECT(adore_create(&c, nullptr, fake, n, nullptr, &h) == ADORE_E_INVALID);
  EXPECT(adore_create(&c, &wt, nullptr, n, nullptr, &h) == ADORE_E_INVALID);
  EXPECT(adore_create(&c, &wt, fake, n - 1, nullptr, &h) == ADORE_E_WORKSPACE);
  EXPECT(adore_create(&c, &wt, static_cast<char *>(fake) + 16, n, nullptr, &h) == ADORE_E_WORKSPACE);
  // every integer field at values around its limits: the layout arithmetic must not overflow or divide by zero
  const int32_t probes[] = {-2147483647 - 1, -1, 0, 1, 2, 7, 63, 64, 65, 1023, 1024, 1025, 65535, 65536, 2147483647};
  for (size_t field = 0; field < 10; ++field) {
    for (int32_t v : probes) {
      adore_config x = tiny();
      reinterpret_cast<int32_t *>(&x)[field] = v;
      const size_t bytes = adore_workspace_bytes(&x);
      adore_ctx *hx = nullptr;
      const int rc = adore_create(&x, &wt, fake, bytes ? bytes : 256, nullptr, &hx);
      EXPECT(rc == ADORE_OK || rc == ADORE_E_INVALID || rc == ADORE_E_UNSUPPORTED || rc == ADORE_E_WORKSPACE);
      if (rc == ADORE_OK) {
        EXPECT(bytes > 0);
        EXPECT(adore_destroy(hx) == ADORE_OK);
      }
    }
  }
  for (int mode = -1; mode <= 3; ++mode) {
    for (float base : {0.f, 10000.f, -1.f}) {
      adore_config x = tiny();
      x.score_mode = mode;
      x.rope_base = base;
      const size_t bytes = adore_workspace_bytes(&x);
      adore_ctx *hx = nullptr;
      const int rc = adore_create(&x, &wt, fake, bytes ? bytes : 256, nullptr, &hx);
      if (rc == ADORE_OK) EXPECT(adore_destroy(hx) == ADORE_OK);
    }
  }
  // one context, calls out of order and with null arguments
  EXPECT(adore_create(&c, &wt, fake, n, nullptr, &h) == ADORE_OK);
  EXPECT(adore_attend(h, 0, fake, fake, fake, ffake) == ADORE_E_STATE);
  { const int rc = adore_attend(h, 5, fake, fake, fake, ffake); EXPECT(rc == ADORE_E_INVALID || rc == ADORE_E_STATE); }
  EXPECT(adore_schedule(h, fake, nullptr, nullptr, nullptr, nullptr) == ADORE_E_STATE);
  EXPECT(adore_rebuild(h, 0, fake) == ADORE_E_STATE);
  EXPECT(adore_decode_step(h, fake, fake, fake, fake, fake, nullptr, ffake, nullptr) == ADORE_E_STATE);
  EXPECT(adore_init_cache(h, fake, fake, fake, fake, nullptr, 0) == ADORE_E_INVALID);
  EXPECT(adore_init_cache(h, fake, fake, fake, fake, nullptr, c.max_positions) == ADORE_E_INVALID);
  EXPECT(adore_init_cache(h, nullptr, fake, fake, fake, nullptr, 4) == ADORE_E_INVALID);
  EXPECT(adore_set_state(h, nullptr, nullptr, nullptr, nullptr, nullptr, 5) == ADORE_E_INVALID);
  EXPECT(adore_set_state(h, static_cast<const int32_t *>(fake), nullptr, nullptr, nullptr, nullptr, 0) == ADORE_E_INVALID);
  EXPECT(adore_set_input_order(nullptr, 0) == ADORE_E_INVALID);
  EXPECT(adore_set_input_order(h, 0) == ADORE_OK);
  EXPECT(adore_set_input_order(h, 1) == ADORE_OK);
  EXPECT(adore_set_timing(h, 1) == ADORE_OK);
  EXPECT(adore_set_timing(h, 0) == ADORE_OK);
  adore_forward_weights fw = {fake, fake};
  EXPECT(adore_forward_step(h, nullptr, fake, nullptr, fake, nullptr, nullptr, nullptr, nullptr) == ADORE_E_INVALID);
  EXPECT(adore_forward_step(h, &fw, fake, nullptr, fake, nullptr, nullptr, nullptr, nullptr) == ADORE_E_STATE);
  int32_t damaged = 7;
  EXPECT(adore_check_guards(h, &damaged) == ADORE_OK && damaged == -1);
  EXPECT(adore_check_guards(h, nullptr) == ADORE_E_INVALID);
  int32_t step = 0;
  EXPECT(adore_get_state(h, nullptr, nullptr, nullptr, nullptr, nullptr, &step) == ADORE_E_STATE);
  EXPECT(adore_destroy(h) == ADORE_OK);
  EXPECT(adore_destroy(nullptr) == ADORE_E_INVALID);
  // a stack called layer by layer keeps to the caller's stream while its inputs are ordered, whenever that is said
  {
    adore_config x = tiny();
    x.layers = 3;
    adore_ctx *hx = nullptr;
    EXPECT(adore_create(&x, &wt, fake, adore_workspace_bytes(&x), nullptr, &hx) == ADORE_OK);
    EXPECT(hx->one_stream);
    EXPECT(adore_set_input_order(hx, 0) == ADORE_OK && !hx->one_stream);
    EXPECT(adore_set_input_order(hx, 1) == ADORE_OK && hx->one_stream);
    EXPECT(adore_destroy(hx) == ADORE_OK);
    // one layer whose selections ride in the attention launch has little to wait for once its inputs are known ahead; as
    // launches of their own they stay where they are
    x = tiny();
    x.dtype = ADORE_BF16; x.batch = 8; x.heads = 16; x.head_dim = 128; x.hidden = 2048; x.cache_slots = 256; x.rebuild_budget = 16;
    EXPECT(adore_create(&x, &wt, fake, adore_workspace_bytes(&x), nullptr, &hx) == ADORE_OK);
    EXPECT(hx->one_stream && hx->one_when[0] && hx->one_when[1]);
    EXPECT(adore_set_input_order(hx, 0) == ADORE_OK && !hx->one_stream && hx->one_when[0]);
    EXPECT(adore_destroy(hx) == ADORE_OK);
  }
  // the choice in parts of 1024 tokens: at most 64 of them, and (parts + 1) R + 1 <= 4096 keys
  for (const int (&v)[3] :
       (const int[][3]){{63, 65537, 1}, {63, 65538, 0}, {64, 63489, 1}, {64, 63490, 0}, {128, 30721, 1}, {128, 30722, 0}, {300, 12289, 1}, {300, 12290, 0}}) {
    adore_config x = tiny();
    x.dtype = ADORE_BF16; x.ctrl_hidden = 128; x.cache_slots = 1024;
    x.rebuild_budget = v[0]; x.max_positions = v[1];
    adore_ctx *hx = nullptr;
    EXPECT(adore_create(&x, &wt, fake, adore_workspace_bytes(&x), nullptr, &hx) == ADORE_OK);
    EXPECT(hx->ride_parts == (v[2] != 0));
    EXPECT(adore_destroy(hx) == ADORE_OK);
  }
  // H2O mode: a step that fails behind its attention, which adds to the scores, is not taken a second time
  for (const int heads : {4, 256}) {   // rows cut into splits, with a release of its own; whole rows, released with the attention
    adore_config x = tiny();
    x.score_mode = ADORE_SCORE_H2O; x.batch = heads / 4; x.cache_slots = 128;
    adore_ctx *hx = nullptr;
    EXPECT(adore_create(&x, &wt, fake, adore_workspace_bytes(&x), nullptr, &hx) == ADORE_OK);
    EXPECT((hx->nsplit == 1) == (heads == 256));
    EXPECT(adore_init_cache(hx, fake, fake, fake, fake, nullptr, 300) == ADORE_OK);
    EXPECT(adore_decode_step(hx, fake, fake, fake, fake, nullptr, nullptr, ffake, nullptr) == ADORE_OK);
    launches = 0;
    failing_launch = heads == 256 ? 2 : 4;   // the choice
    EXPECT(adore_decode_step(hx, fake, fake, fake, fake, nullptr, nullptr, ffake, nullptr) == ADORE_E_HIP);
    failing_launch = -1;
    EXPECT(adore_decode_step(hx, fake, fake, fake, fake, nullptr, nullptr, ffake, nullptr) == ADORE_E_STATE);
    EXPECT(adore_init_cache(hx, fake, fake, fake, fake, nullptr, 300) == ADORE_OK);
    EXPECT(adore_decode_step(hx, fake, fake, fake, fake, nullptr, nullptr, ffake, nullptr) == ADORE_OK);
    EXPECT(adore_destroy(hx) == ADORE_OK);
  }
  // A prompt's chunks in the halves of a copy that lies in the cache: a short last one, whose projection is cut into slices, stays in
  // its half (the other one is being read meanwhile).  34 chunks of 520 tokens and one of 241; 33 and one of 250 in the upper half; 49 and
  // one of 122 of two sequences.
  setenv("ADORE_NO_OVERLAP", "1", 1);   // (no streams to be made; the chunks and their copies are the same)
  for (const int (&v)[4] : (const int[][4]){{1, 780, 17921, 4096}, {1, 780, 17921, 2048}, {1, 780, 17410, 4096}, {2, 780, 25602, 2048}}) {
    adore_config x = tiny();
    x.dtype = ADORE_BF16; x.ctrl_hidden = 128; x.heads = 8; x.head_dim = 128; x.rebuild_budget = 8;
    x.batch = v[0]; x.cache_slots = v[1]; x.max_positions = v[2] + 8; x.hidden = v[3];
    adore_ctx *hx = nullptr;
    EXPECT(adore_create(&x, &wt, fake, adore_workspace_bytes(&x), nullptr, &hx) == ADORE_OK);
    EXPECT(hx->gi_rows[2] * 2 == hx->gi_rows[1] && hx->gi_rows[1] < size_t(v[0]) * v[2]);
    sliced.clear();
    EXPECT(adore_init_cache(hx, fake, fake, fake, fake, nullptr, v[2]) == ADORE_OK);
    EXPECT(!sliced.empty());
    for (const SlicedProjection &p : sliced) {
      EXPECT(p.gi == hx->gi[1] || p.gi == hx->gi[2]);
      EXPECT(p.width == 384 && size_t(p.slices) * p.tokens <= hx->gi_rows[2]);
    }
    EXPECT(adore_destroy(hx) == ADORE_OK);
  }
  unsetenv("ADORE_NO_OVERLAP");
  // the debug layout
  setenv("ADORE_GUARD_WORDS", "1", 1);
  const size_t guarded = adore_workspace_bytes(&c);
  EXPECT(guarded > n && (guarded - n) % 256 == 0);
  EXPECT(adore_create(&c, &wt, fake, n, nullptr, &h) == ADORE_E_WORKSPACE);
  EXPECT(adore_create(&c, &wt, fake, guarded, nullptr, &h) == ADORE_OK);
  EXPECT(adore_destroy(h) == ADORE_OK);
  unsetenv("ADORE_GUARD_WORDS");
  // tables
  for (int code : {0, -1, -2, -3, -4, -5, -99, 12345}) EXPECT(adore_strerror(code) != nullptr && std::strlen(adore_strerror(code)) > 0);
  for (int i = -3; i < ADORE_N_KERNELS + 3; ++i) EXPECT(adore_kernel_name(i) != nullptr);
  // top-K attention: sizes and argument checks
  EXPECT(adore_topk_attention_workspace_bytes(0, 8, 64) == 0);
  EXPECT(adore_topk_attention_workspace_bytes(3, 100, 128) == size_t(3) * 128 * 128 * 2);
  for (int32_t rows : {1, 7, 512, 65535, 65536, 2147483647})
    for (int32_t seq : {1, 31, 32, 33, 2048, 2049, 32768, 32769, 2147483647})
      (void)adore_topk_attention_workspace_bytes(rows, seq, 128);
  const size_t tn = adore_topk_attention_workspace_bytes(2, 64, 64);
  EXPECT(adore_topk_attention(nullptr, fake, fake, fake, fake, tn, 2, 64, 64, 4, nullptr) == ADORE_E_INVALID);
  EXPECT(adore_topk_attention(fake, fake, fake, fake, fake, tn, 2, 64, 64, 0, nullptr) == ADORE_E_INVALID);
  EXPECT(adore_topk_attention(fake, fake, fake, fake, fake, tn, 2, 64, 96, 4, nullptr) == ADORE_E_UNSUPPORTED);
  EXPECT(adore_topk_attention(fake, fake, fake, fake, fake, tn - 1, 2, 64, 64, 4, nullptr) == ADORE_E_WORKSPACE);
  EXPECT(adore_topk_attention_static(fake, fake, fake, nullptr, 2, 64, 64, 4, nullptr) == ADORE_E_INVALID);
  EXPECT(adore_topk_attention_static(fake, fake, fake, fake, 2, 4096, 64, 4, nullptr) == ADORE_E_WORKSPACE);
  EXPECT(adore_topk_attention_static(fake, fake, fake, fake, 60000, 2048, 128, 4, nullptr) == ADORE_E_WORKSPACE);
  // ... and the sizes of its launches: HIP takes fewer than 2^32 threads, and every block of queries has its workgroup
  for (int32_t rows : {1, 15, 512, 16385, 65535})
    for (int32_t seq : {1, 64, 65, 8192, 8193, 16500, 32768})
      for (int32_t d : {64, 128}) {
        launched_grid.clear();
        launched_block.clear();
        const size_t bytes = adore_topk_attention_workspace_bytes(rows, seq, d);
        EXPECT(adore_topk_attention(fake, fake, fake, fake, fake, bytes, rows, seq, d, 96, nullptr) == ADORE_OK);
        uint64_t groups = 0;
        for (size_t i = 0; i < launched_grid.size(); ++i) {
          EXPECT(uint64_t(launched_grid[i].x) * launched_block[i].x < (uint64_t(1) << 32));
          EXPECT(launched_block[i].x == launched_block[0].x && launched_grid[i].y == 1 && launched_grid[i].z == 1);
          groups += launched_grid[i].x;
        }
        EXPECT(!launched_grid.empty());
        // blocks of 64 queries where they fill the compute units, else of 32; four waves either way
        const int32_t queries = int64_t(rows) * ((seq + 63) / 64) < (d == 128 ? 256 : 512) ? 32 : 64;
        EXPECT(!launched_block.empty() && launched_block[0].x == 256);
        EXPECT(groups == uint64_t(rows) * ((seq + queries - 1) / queries));
      }
  if (failures) {
    std::fprintf(stderr, "%d unexpected answers\n", failures);
    return 1;
  }
  std::puts("host checks ok");
  return 0;
}
