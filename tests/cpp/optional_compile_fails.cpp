// Registers an op graph (a transpose, then a row reduce of its result) while the device compile of the
// row reduce's second module -- the one that reads the transpose's operand itself -- fails: the
// registration has to succeed, the graph runs as two kernels.  Registered again, nothing is compiled.
//
// usage: optional_compile_fails <graph file>   int32 n_ops, int32 n_cs, int32 n_dims, the records.
// Prints "compiles=<n> failed=<k> again=<m>".
#include <dlfcn.h>
#include <hip/hiprtc.h>

#include <cstdio>
#include <cstring>
#include <vector>

#include "disc.h"

static bool g_fail = false;      // the program that was created last is the optional one
static int g_failed = 0;
extern "C" hiprtcResult hiprtcCreateProgram(hiprtcProgram* prog, const char* src, const char* name, int n, const char* const* headers,
                                            const char* const* names) {
  typedef hiprtcResult (*Fn)(hiprtcProgram*, const char*, const char*, int, const char* const*, const char* const*);
  g_fail = strstr(src, "xp_src(const Args& A) { return") != nullptr;
  return ((Fn)dlsym(RTLD_NEXT, "hiprtcCreateProgram"))(prog, src, name, n, headers, names);
}
extern "C" hiprtcResult hiprtcCompileProgram(hiprtcProgram prog, int n, const char* const* options) {
  typedef hiprtcResult (*Fn)(hiprtcProgram, int, const char* const*);
  if (g_fail) {
    ++g_failed;
    return HIPRTC_ERROR_COMPILATION;
  }
  return ((Fn)dlsym(RTLD_NEXT, "hiprtcCompileProgram"))(prog, n, options);
}

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  FILE* f = fopen(argv[1], "rb");
  if (!f) return 3;
  int32_t hdr[3];
  if (fread(hdr, 4, 3, f) != 3) return 3;
  std::vector<disc_op> ops(hdr[0]);
  std::vector<disc_constraint> cs(hdr[1] > 0 ? hdr[1] : 1);
  if (fread(ops.data(), sizeof(disc_op), hdr[0], f) != (size_t)hdr[0]) return 3;
  if (hdr[1] > 0 && fread(cs.data(), sizeof(disc_constraint), hdr[1], f) != (size_t)hdr[1]) return 3;
  fclose(f);
  disc_ctx* ctx = nullptr;
  if (disc_create(&ctx, -1) != DISC_OK) return 4;
  disc_stats_t first, second;
  int32_t id = -1;
  if (disc_register_graph(ctx, ops.data(), hdr[0], cs.data(), hdr[1], &id) != DISC_OK) {
    fprintf(stderr, "%s\n", disc_last_error(ctx));
    return 5;
  }
  disc_get_stats(ctx, &first);
  if (disc_register_graph(ctx, ops.data(), hdr[0], cs.data(), hdr[1], &id) != DISC_OK) return 6;
  disc_get_stats(ctx, &second);
  printf("compiles=%d failed=%d again=%d\n", (int)first.compile_events, g_failed, (int)(second.compile_events - first.compile_events));
  disc_destroy(ctx);
  return 0;
}
