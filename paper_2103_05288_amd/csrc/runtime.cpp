// Context, pattern cache, the one device compile per pattern, and the launch path.
//
// The launch path is the "generated runtime flow" of the paper (Section 4.2) in the form of a
// closure specialised at registration: shape calculation from the runtime dims, the check of
// the registered equalities, version and launch-dimension selection (Section 4.3), filling of
// the kernel-argument block, one enqueue.  It walks recipes made of a handful of integer
// products and comparisons; the op list of the pattern is never visited at launch time.
#include <hip/hip_runtime_api.h>
#include <hip/hiprtc.h>

#include <chrono>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <numeric>
#include <set>
#include <sstream>

#include "disc_internal.hpp"

namespace disc {

extern const char* const kDeviceHeader;   // disc_device.h, embedded at build time

namespace {

struct DeviceRowPlan {   // mirrors disc::RowPlan of the device header
  int32_t G, log2G, nv, flags, rpb;
};
struct DeviceColPlan {   // mirrors disc::ColPlan of the device header
  int32_t GC, log2GC, nchunk, lists;
  int64_t chunk_rows, outer, epi_rows;
};
constexpr int kLdsStep = 512, kLdsSteps = 64 * 1024 / kLdsStep + 2;
constexpr int kArgBufBytes = 4096;    // kernel-argument block + launch-plan struct
constexpr int kMaxShapeValues = 64;   // strides + base offsets + padding windows of one pattern
struct FastDivHost {
  uint32_t d, m, s, pad;
};

FastDivHost make_fastdiv(uint64_t d) {
  FastDivHost f{1, 1, 0, 0};
  if (d == 0 || d > 0x7fffffffull) { f.d = (uint32_t)(d > 0xffffffffull ? 0xffffffffu : d); return f; }
  uint32_t s = 0;
  while ((1ull << s) < d) ++s;
  f.d = (uint32_t)d;
  f.s = s;
  f.m = (uint32_t)((((1ull << s) - d) << 32) / d + 1);
  return f;
}

struct Pattern {
  Analysis an;
  Generated gen;
  std::string key;
  int compile_events = 0;
  double compile_ms = 0;
  hipModule_t module = nullptr;
  // Launch-time tables, indexed by kernel number: nothing on the launch path looks up a name.
  hipFunction_t fn[K_COUNT] = {};
  // blocks resident per CU by (kernel, block-size class, dynamic LDS in steps of kLdsStep bytes),
  // asked from the runtime on first use (0 = not asked yet)
  mutable int16_t resident[K_COUNT][3][kLdsSteps] = {};
  bool is_static = false;                             // module specialised for static_dims only
  std::vector<int64_t> static_dims;
  // constraint recipes
  std::vector<std::pair<int, int>> eq_checks;         // symbolic dims that must be equal
  std::vector<std::pair<int, int64_t>> static_checks; // symbolic dim that must equal a static size
  std::vector<int> class_of_dim;
  int n_classes = 0;
  // element count recipes for algorithmic bytes
  std::vector<std::pair<DimProduct, int>> io_numel;   // (numel product, bytes per element)
};

struct ShapeVals {
  int64_t group[4] = {1, 1, 1, 1};
  int64_t rows = 1, inner = 1, mid = 0;
  int64_t products[kMaxShapeValues];   // strides, base offsets, padding windows (no allocation at launch)
  int64_t alg_bytes = 0;
};

bool mul_ovf(int64_t a, int64_t b, int64_t* r) { return __builtin_mul_overflow(a, b, r); }

bool eval_product(const DimProduct& p, const int64_t* dims, int64_t* out) {
  int64_t v = p.stat;
  for (int s : p.sym)
    if (mul_ovf(v, dims[s], &v)) return false;
  *out = v;
  return true;
}

int64_t now_ns() {
  return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

}  // namespace
}  // namespace disc

using namespace disc;

// ---- op graphs larger than one fusion pattern (Section 4.3, fusion decision over a graph) -------
struct GraphGroup {
  std::vector<int> ops;          // graph op ids fused into this pattern, in graph order
  int pattern_id = -1;
  std::vector<int> in_values;    // graph value ids bound to the pattern's PARAMs, in order
  std::vector<int> out_values;   // graph value ids produced by the pattern's OUTPUTs, in order
  // where each of those values lives at launch, resolved at registration: (kind, index) with kind
  // 0 = graph input, 1 = graph output, 2 = planned buffer
  std::vector<std::pair<int, int>> in_place, out_place;
  // a row reduce that takes the result of the transpose pattern in front of it: the module whose kernels read
  // the transpose's operand themselves (index into disc_ctx::fused, -1: none), and which input that is
  int fused = -1, fused_input = -1;
};
struct GraphIntermediate {
  int value = -1;                // produced by group `first`, last read by group `last`
  int first = 0, last = 0;
  int buffer = -1;
};
struct Graph {
  std::vector<disc_op> ops;
  std::vector<disc_constraint> cs;
  std::vector<int> group_of_op;  // -1 for leaves and OUTPUT ops
  std::vector<char> remat;       // value is recomputed by the patterns that read it instead of crossing a cut
  std::vector<char> needed;      // some graph output depends on the op (the others are dead code)
  std::vector<GraphGroup> groups;
  std::vector<GraphIntermediate> inter;
  std::map<int, int> inter_of_value;
  std::vector<int> buffer_value;         // a value whose size every tenant of the buffer shares
  std::map<int, int> param_index;        // PARAM op id -> input index
  std::map<int, int> output_index;       // value id -> output index (graph OUTPUT ops)
  int n_sym = 0, n_inputs = 0, n_outputs = 0;
};

struct disc_ctx {
  std::vector<std::unique_ptr<Graph>> graphs;
  int device = -1;
  int n_cus = 256;
  std::string err;
  std::vector<std::unique_ptr<Pattern>> patterns;
  std::vector<std::unique_ptr<Pattern>> fused;   // row reduces of op graphs that take an operand transposed ...
  std::map<std::pair<int, int>, int> fused_of;   // ... by pattern and input: compiled once, shared by all graphs (-1: it could not be)
  std::map<std::string, int> cache;
  disc_stats_t stats{};
  int force_variant = -1;
  hipModule_t util_module = nullptr;
  hipFunction_t util_copy = nullptr, util_copy_nt = nullptr, util_empty = nullptr;
  hipFunction_t util_mix[2][2][4] = {};   // [kind][non-temporal][log2 slots in flight]
  // test overrides (disc_test_option); the defaults are the host rules
  int row_nt = -1;           // non-temporal versions: -1 = host rule, 0 = never, 1 = wherever the version exists
  int row_rounds = 0;        // row kernels: grid = this many rounds of resident blocks (0: host rule)
  int row_stage = 1;         // 0: row vectors are never staged in LDS
  int compact_looks = -1;    // compaction in one pass: looks for a count (-1: host rule)
  int row_shift = 1;         // 0: vector slots of ragged rows are never shifted to the tensor's 16-byte boundaries
};
constexpr int kGridMult = 8;     // loop / column kernels: grid capped at this many blocks per CU
constexpr int kLoopUnroll = 4;   // loop kernels: slots in flight per lane

namespace {

int set_err(disc_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}

int hip_fail(disc_ctx* c, hipError_t e, const char* what) {
  return set_err(c, DISC_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

int compile_source(disc_ctx* c, const std::string& src, std::vector<char>* code, double* ms) {
  hiprtcProgram prog;
  if (hiprtcCreateProgram(&prog, src.c_str(), "disc_pattern.hip", 0, nullptr, nullptr) != HIPRTC_SUCCESS)
    return set_err(c, DISC_ERR_COMPILE, "hiprtcCreateProgram failed");
  std::vector<const char*> opts = {"--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                                   "-packed-fp32-ops", "-Wno-unused-value",
                                   // the fused expressions are scalar per element on purpose: no packed-fp32 pairs
                                   "-fno-slp-vectorize", "-fno-vectorize"};
  auto t0 = std::chrono::steady_clock::now();
  hiprtcResult r = hiprtcCompileProgram(prog, (int)opts.size(), opts.data());
  *ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  if (r != HIPRTC_SUCCESS) {
    size_t n = 0;
    hiprtcGetProgramLogSize(prog, &n);
    std::string log(n, '\0');
    if (n) hiprtcGetProgramLog(prog, &log[0]);
    hiprtcDestroyProgram(&prog);
    return set_err(c, DISC_ERR_COMPILE, "device compile failed:\n" + log);
  }
  size_t n = 0;
  hiprtcGetCodeSize(prog, &n);
  code->resize(n);
  hiprtcGetCode(prog, code->data());
  hiprtcDestroyProgram(&prog);
  return DISC_OK;
}

Pattern* get_pattern(disc_ctx* c, int32_t id) {
  if (!c || id < 0 || id >= (int)c->patterns.size()) return nullptr;
  return c->patterns[id].get();
}

// ---- shape calculation (host) -------------------------------------------------------------
int shape_calc(disc_ctx* c, const Pattern& p, const int64_t* dims, int n_dims, ShapeVals* sv) {
  if (!dims && p.an.n_sym > 0) return set_err(c, DISC_ERR_INVALID_ARG, "dims is null");
  if (n_dims != p.an.n_sym) {
    char buf[96];
    snprintf(buf, sizeof buf, "pattern has %d symbolic dims, %d given", p.an.n_sym, n_dims);
    return set_err(c, DISC_ERR_INVALID_ARG, buf);
  }
  for (int i = 0; i < n_dims; ++i)
    if (dims[i] < 0) return set_err(c, DISC_ERR_SHAPE, "negative dimension");
  char buf[160];
  for (const auto& e : p.eq_checks)
    if (dims[e.first] != dims[e.second]) {
      snprintf(buf, sizeof buf, "dims[%d] = %lld and dims[%d] = %lld were registered as equal", e.first,
               (long long)dims[e.first], e.second, (long long)dims[e.second]);
      return set_err(c, DISC_ERR_CONSTRAINT, buf);
    }
  for (const auto& e : p.static_checks)
    if (dims[e.first] != e.second) {
      snprintf(buf, sizeof buf, "dims[%d] = %lld must equal the static size %lld", e.first, (long long)dims[e.first],
               (long long)e.second);
      return set_err(c, DISC_ERR_CONSTRAINT, buf);
    }
  const Analysis& an = p.an;
  const int ng = (int)an.groups.size();
  int64_t total = 1;
  for (int g = 0; g < ng; ++g) {
    if (!eval_product(an.group_size[g], dims, &sv->group[g]) || mul_ovf(total, sv->group[g], &total))
      return set_err(c, DISC_ERR_SHAPE, "element count overflows int64");
  }
  for (const auto& nc : an.numel_checks) {
    int64_t n = 0;
    if (!eval_product(nc.second, dims, &n)) return set_err(c, DISC_ERR_SHAPE, "element count overflows int64");
    if (n != total) {
      snprintf(buf, sizeof buf, "op %d has %lld elements, the iteration space %lld: they were registered as equal in size",
               nc.first, (long long)n, (long long)total);
      return set_err(c, DISC_ERR_CONSTRAINT, buf);
    }
  }
  sv->inner = sv->group[an.inner_group];
  sv->rows = 1;
  for (int g = 0; g < an.inner_group; ++g) sv->rows *= sv->group[g];
  sv->mid = an.mid_group >= 0 ? sv->group[an.mid_group] : 0;
  for (size_t i = 0; i < an.products.size(); ++i)
    if (!eval_product(an.products[i], dims, &sv->products[i]))
      return set_err(c, DISC_ERR_SHAPE, "stride overflows int64");
  // sliced operands (Section 4.1: slice starts are runtime values): bounds, then base offsets
  auto dim_val = [&](int32_t d) { return d >= 0 ? dims[d] : -(int64_t)d; };
  auto start_val = [&](int32_t s) { return s >= 0 ? dims[s] : (int64_t)(-1 - s); };
  for (const auto& sc : an.slice_checks) {
    const int64_t st = start_val(sc.start), n = dim_val(sc.size_dim), ext = dim_val(sc.src_dim);
    if (st < 0 || n > ext || st > ext - n) {
      snprintf(buf, sizeof buf, "op %d (%s), axis %d: [%lld, %lld) does not fit the extent %lld", sc.op,
               an.ops[sc.op].opcode == DISC_PAD ? "pad" : "slice", sc.axis, (long long)st, (long long)(st + n), (long long)ext);
      return set_err(c, DISC_ERR_SHAPE, buf);
    }
  }
  for (size_t i = 0; i < an.offsets.size(); ++i) {
    int64_t sum = 0;
    for (const auto& t : an.offsets[i].terms) {
      int64_t stride = 0, term = 0;
      if (!eval_product(t.second, dims, &stride) || mul_ovf(stride, start_val(t.first), &term) ||
          __builtin_add_overflow(sum, term, &sum))
        return set_err(c, DISC_ERR_SHAPE, "slice offset overflows int64");
    }
    sv->products[an.products.size() + i] = sum;
  }
  for (size_t i = 0; i < an.windows.size(); ++i) {
    const WindowRecipe& w = an.windows[i];
    int64_t inner = 0, lo = 0, hi = 0;
    if (!eval_product(w.inner_sizes, dims, &inner) || mul_ovf(start_val(w.low), inner, &lo) ||
        mul_ovf(start_val(w.low) + dim_val(w.extent_dim), inner, &hi))
      return set_err(c, DISC_ERR_SHAPE, "padding window overflows int64");
    sv->products[an.products.size() + an.offsets.size() + 2 * i] = lo;
    sv->products[an.products.size() + an.offsets.size() + 2 * i + 1] = hi;
  }
  sv->alg_bytes = 0;
  for (const auto& io : p.io_numel) {
    int64_t n = 0;
    if (!eval_product(io.first, dims, &n) || mul_ovf(n, io.second, &n))
      return set_err(c, DISC_ERR_SHAPE, "tensor size overflows int64");
    sv->alg_bytes += n;
  }
  return DISC_OK;
}

int ilog2_ceil(int64_t v) {
  int l = 0;
  while ((1ll << l) < v) ++l;
  return l;
}

struct LaunchRec {
  int kid = -1;              // KernelId
  uint32_t grid[3] = {1, 1, 1};
  uint32_t block = 256;
  int plan_kind = 0;         // 0 none, 1 RowPlan, 2 ColPlan
  uint32_t dyn_lds = 0;      // dynamic LDS bytes
  DeviceRowPlan rp{};
  DeviceColPlan cp{};
};

struct FullPlan {
  disc_plan_t pub{};
  ShapeVals sv;
  LaunchRec launches[3];
  int64_t nslots = 0, spr = 0;
  int64_t aux[4] = {0, 0, 0, 0};
  size_t ws_off[2] = {0, 0};
  size_t ws_need = 0;        // what this launch uses; pub.workspace_bytes covers every alignment of the operands
};

// Loop-fusion launch geometry for an iteration space [rows, inner]; shared by loop patterns and
// by the epilogue stage of column reduces.  want_vec / want_i64: -1 = let the shape decide.
// Launches that move less than this may be read back from the memory-side cache (256 MB) by
// whatever kernel consumes the result; the non-temporal versions are kept for larger ones, which
// stream through the caches anyway.
constexpr int64_t kNonTemporalMinBytes = 64ll << 20;
// Ragged rows with the non-temporal hint: fewest lanes per row, rows off dword boundaries / others.
constexpr int kMinLinesG = 64, kMinLinesEvenG = 128;
constexpr int64_t kNarrowShiftMinBytes = kNonTemporalMinBytes * 5 / 4;
// LDS for row vectors, and for their copies that shifted slots read in wide blocks of large launches.
constexpr int64_t kMaxStageBytes = 48 * 1024, kMaxShiftedStageBytes = 64 * 1024;
// Tile transposes: from this many tiles on no lists, whose four tile rows of as many tiles, in one row of tiles, would not be counted in 32 bits.
constexpr int64_t kTransposeListTiles = 1ll << 29;
// Compaction: from this many tiles on (2^17 i32 elements), two launches instead of three: the blocks of
// the scatter launch add up the counts in front of them by themselves (14 us a call against 15-16 at
// 2^17 .. 2^20 elements, where the launches are what is paid for), in at most kCompactBlocksPerCu blocks to a CU.
// From kCompactOnePassMinBytes on -- the line of the non-temporal versions, which its stores are -- one pass (the kernel's comment
// has both sides; 8 x 10^6 i32 20.5 / 17.1, 4 x 10^6 12.6 / 9.6, 6 x 10^6 and 3 x 10^6 i64 the same); from kCompactStreamMinBytes on
// the kept values are non-temporal too.  A look at a missing count takes 2 us: the limit is a millisecond, far beyond the time
// between two blocks that are both resident.
constexpr int64_t kCompactTwoLaunchTiles = 32, kCompactBlocksPerCu = 4;
constexpr int64_t kCompactOnePassMinBytes = kNonTemporalMinBytes, kCompactStreamMinBytes = 150ll << 20, kCompactLooks = 500;

// nt_name: the non-temporal sibling of names[0] (vector width, 32-bit index), taken for large
// launches (`big`) whose rows start on 16-byte boundaries (`aligned`: the full-size operands are;
// inner a multiple of the width).
int plan_loop(disc_ctx* c, int64_t rows, int64_t inner, int V, int want_vec, int want_i64, const int names[4],
              int nt_name, bool aligned, bool big, FullPlan* fp, LaunchRec* L, bool* vec_out, bool* i64_out) {
  bool vec;
  {
    const int64_t spr_v = (inner + V - 1) / V;
    const double waste = 1.0 - (double)inner / (double)(spr_v * V);
    vec = waste <= 0.25;
  }
  if (want_vec >= 0) vec = want_vec != 0;
  const int v = vec ? V : 1;
  int64_t spr = (inner + v - 1) / v, nslots;
  if (mul_ovf(spr, rows, &nslots)) return set_err(c, DISC_ERR_SHAPE, "slot count overflows int64");
  bool i64 = nslots >= (1ll << 31) - (1ll << 24) || inner >= (1ll << 31) - 16 || rows >= (1ll << 31);
  if (want_i64 == 1) i64 = true;
  else if (want_i64 == 0 && i64) return set_err(c, DISC_ERR_INVALID_ARG, "forced 32-bit version cannot index this shape");
  const int U = i64 ? 1 : kLoopUnroll;
  const int64_t max_grid = (int64_t)c->n_cus * kGridMult;
  int64_t blocks = (nslots + 256ll * U - 1) / (256ll * U);
  blocks = std::min(blocks, i64 ? max_grid * 4 : max_grid);
  L->kid = names[(vec ? 0 : 2) + (i64 ? 1 : 0)];
  if (nt_name >= 0 && vec && v > 1 && !i64 && aligned && inner % v == 0 && c->row_nt != 0 &&
      (c->row_nt > 0 || big))
    L->kid = nt_name;
  L->grid[0] = (uint32_t)blocks;
  L->block = 256;
  fp->nslots = nslots;
  fp->spr = spr;
  fp->pub.index_bits = i64 ? 64 : 32;
  fp->pub.vec_width = v;
  fp->pub.slots_per_lane = U;
  *vec_out = vec;
  *i64_out = i64;
  return DISC_OK;
}

// Blocks of a kernel that one CU holds at a given block size and dynamic LDS size, as the
// runtime computes it from the compiled kernel's register and LDS use (asked once per
// combination).  Without a device: an estimate from a 16-wavefront budget.
int resident_blocks(const disc_ctx* c, const Pattern& p, int kid, uint32_t block, uint32_t dyn_lds);

// ---- version + launch-dimension selection (host) ---------------------------------------------
// ws_limit: where a plan can do with less workspace than it would like, what it may use.
int make_plan(disc_ctx* c, const Pattern& p, const int64_t* dims, int n_dims, int force, const void* const* inputs,
              void* const* outputs, FullPlan* fp, size_t ws_limit = SIZE_MAX) {
  // pointer values: wide accesses need element alignment only; the non-temporal row versions are
  // picked for 16-byte aligned full-size operands (null arrays: assumed aligned)
  if (p.is_static) {
    if (force >= 0) return set_err(c, DISC_ERR_INVALID_ARG, "a single-shape pattern has one kernel version");
    if (n_dims != (int)p.static_dims.size() || !std::equal(dims, dims + n_dims, p.static_dims.begin()))
      return set_err(c, DISC_ERR_SHAPE, "pattern was compiled for one shape and is launched with another");
  }
  int rc = shape_calc(c, p, dims, n_dims, &fp->sv);
  if (rc) return rc;
  // every full-size operand on a 16-byte boundary (null pointer arrays: assumed)
  auto full_aligned = [&]() {
    for (const Access& a : p.an.accesses) {
      if (a.kind != ACC_FULL) continue;
      const void* ptr = a.is_output ? (outputs ? outputs[a.slot] : nullptr) : (inputs ? inputs[a.slot] : nullptr);
      if (reinterpret_cast<uintptr_t>(ptr) % 16 != 0) return false;
    }
    return true;
  };
  const Analysis& an = p.an;
  const ShapeVals& sv = fp->sv;
  disc_plan_t& pub = fp->pub;
  pub.rows = sv.rows;
  pub.inner = sv.inner;
  pub.mid = sv.mid;
  pub.algorithmic_bytes = sv.alg_bytes;
  pub.workspace_bytes = 0;
  pub.n_launches = 0;
  pub.variant = -1;
  const int V = an.vec_width;
  const int64_t max_grid = (int64_t)c->n_cus * kGridMult;

  if (an.tmpl == DISC_TEMPLATE_TRANSPOSE) {
    if (sv.rows == 0 || sv.inner == 0) return DISC_OK;
    if (force >= 0 && force != DISC_V_TRANSPOSE_TILE)
      return set_err(c, DISC_ERR_INVALID_ARG, "forced version does not belong to a transpose pattern");
    const int ng = (int)an.groups.size();
    const int64_t P = sv.group[ng - 2], Q = sv.group[ng - 1], batch = ng == 3 ? sv.group[0] : 1;
    // tiles of 256 bytes per row: 128 x 128 elements of one or two bytes, 64 x 64 wider ones
    const int64_t ts = dtype_bytes(an.accesses[0].dtype) <= 2 ? 128 : 64;
    int64_t ntiles = batch * ((P + ts - 1) / ts) * ((Q + ts - 1) / ts);
    // two-byte elements: half tiles (64 result columns, see the kernel) for operand and result of up to 84 MiB together, where
    // more tiles in flight count (us, whole / half tiles: 4000 x 4001, 61 MiB, 16.4 / 14.4), and up to 128 MiB where the result's
    // rows start on 32-byte boundaries (8000 x 3700 31.2 / 27.7, 14400 x 2001 28.5 / 24.8, 6000 x 4097 25.1 / 24.8; elsewhere a
    // half tile's row ends inside a sector of memory twice as often: 1586 x 15009 28.3 / 32.2, 4264 x 5864 29.1 / 31.4; 37 x
    // 112 x 7877 34.7 / 40.9); and where a whole tile would be half empty: up to 64 result columns (64 x 500000 29.4 / 26.1, 30
    // x 2000000 90.6 / 83.3) or 128 result rows (510230 x 102 106.8 / 88.8, 600000 x 80 52.7 / 41.0; but 102 x 510230 59 / 84)
    const bool half = dtype_bytes(an.accesses[0].dtype) == 2 &&
                      (sv.alg_bytes < (84ll << 20) || (sv.alg_bytes < 2 * kNonTemporalMinBytes && Q % 16 == 0 && Q > 128) || P <= 128 || Q <= 64);
    if (half) ntiles = batch * ((P + 127) / 128) * ((Q + 63) / 64);
    LaunchRec& L = fp->launches[0];
    L.kid = half ? K_TRANSPOSE_TILE_H : K_TRANSPOSE_TILE;
    L.block = 256;
    // A tile to a block (before / after, 8 blocks a CU that walked the tiles: 16384 x 8192 117 / 109, 8192 x 4096 f32 59.1 / 53.1,
    // 9000 x 9000 with lists 87 / 76.4), as many as a launch may have.
    L.grid[0] = (uint32_t)std::min<int64_t>(ntiles, 1 << 23);
    // The order of the tiles: lists where the lines of the operand are shared by tiles that are not of one row either, and
    // for large operands whose rows are whole lines (us, diagonal / lists: 16384 x 8192 109 / 100, 2001 x 28800 63.4 / 54.4, 8192 x
    // 8192 57.2 / 55.7, 14400 x 14400 169 / 167; but 2001 x 14400 27.6 / 30.7, 6400 x 6400 33.6 / 35.5, 4000 x 4000 f32 26.0 / 27.4).
    const bool whole_lines = P * dtype_bytes(an.accesses[0].dtype) % 128 == 0;
    fp->aux[0] = ntiles < kTransposeListTiles && (!whole_lines || sv.alg_bytes >= (192ll << 20));
    pub.variant = DISC_V_TRANSPOSE_TILE;
    pub.n_launches = 1;
    pub.vec_width = 1;
    pub.index_bits = 64;
  } else if (an.tmpl == DISC_TEMPLATE_COMPACT) {
    if (force >= 0 && force != DISC_V_COMPACT_VEC && force != DISC_V_COMPACT_SCALAR)
      return set_err(c, DISC_ERR_INVALID_ARG, "forced version does not belong to a compaction pattern");
    bool vec = V > 1;
    if (force >= 0) vec = force == DISC_V_COMPACT_VEC;
    const int v = vec ? V : 1;
    const int64_t tile = 256ll * kCompactLaneSlots * v;
    const int64_t nb = (sv.inner + tile - 1) / tile;
    const bool two = nb >= kCompactTwoLaunchTiles;
    const bool nt = vec && two && c->row_nt != 0 && (c->row_nt > 0 || sv.alg_bytes >= kNonTemporalMinBytes);
    const bool one_pass = vec && two && p.gen.compact_chain && (c->compact_looks >= 0 || (nt && sv.alg_bytes >= kCompactOnePassMinBytes));
    // three launches: a tile to a block, 8 bytes each; two: runs of parts (a wavefront's share of a tile) as even as can be,
    // four bytes for each wavefront; one pass: four bytes for each tile
    const int64_t parts = (sv.inner + tile / 4 - 1) / (tile / 4);
    const int64_t chunks = one_pass || !two ? nb : std::min<int64_t>(nb, (int64_t)c->n_cus * kCompactBlocksPerCu);
    fp->aux[0] = chunks;
    if (one_pass) {
      fp->aux[1] = 0;
      fp->aux[2] = c->compact_looks >= 0 ? c->compact_looks : kCompactLooks;
      fp->aux[3] = sv.alg_bytes >= kCompactStreamMinBytes;
    } else {
      fp->aux[1] = two ? parts / (4 * chunks) : 1;
      fp->aux[2] = two;
      fp->aux[3] = two ? parts % (4 * chunks) : 0;
    }
    fp->ws_off[0] = 0;
    // (one pass: no less than shorter inputs need, so that a workspace asked for at the most elements serves them all)
    fp->ws_need = one_pass ? (size_t)nb * 4 : two ? (size_t)chunks * 16 : (size_t)std::max<int64_t>(nb, 1) * 8;
    pub.workspace_bytes = one_pass ? std::max(fp->ws_need, (size_t)c->n_cus * kCompactBlocksPerCu * 16) : fp->ws_need;
    pub.variant = vec ? DISC_V_COMPACT_VEC : DISC_V_COMPACT_SCALAR;
    pub.vec_width = v;
    pub.index_bits = 64;
    pub.slots_per_lane = kCompactLaneSlots;
    const uint32_t grid = (uint32_t)std::min<int64_t>(chunks, max_grid * 4);
    int l = 0;
    if (one_pass) {
      // as many blocks as are resident, the same number on every CU
      const int64_t per_cu = std::min<int64_t>(kCompactBlocksPerCu, resident_blocks(c, p, K_COMPACT_CHAIN_VEC, 256, 0));
      fp->launches[0].kid = K_COMPACT_CLEAR;
      fp->launches[0].grid[0] = (uint32_t)((nb + 255) / 256);
      fp->launches[1].kid = K_COMPACT_CHAIN_VEC;
      fp->launches[1].grid[0] = (uint32_t)std::min<int64_t>(nb, std::min<int64_t>((int64_t)c->n_cus * per_cu, 1024));
      l = 2;
    } else if (nb > 0) {
      fp->launches[l].kid = vec ? K_COMPACT_COUNT_VEC : K_COMPACT_COUNT_SCALAR;
      fp->launches[l].grid[0] = grid;
      ++l;
    }
    if (!two) {   // (an empty input still runs the scan launch: it stores the count, zero)
      fp->launches[l].kid = K_COMPACT_SCAN;
      fp->launches[l].block = 1024;
      fp->launches[l].grid[0] = 1;
      ++l;
    }
    if (nb > 0 && !one_pass) {
      fp->launches[l].kid = nt ? K_COMPACT_SCATTER_VEC_NT : vec ? K_COMPACT_SCATTER_VEC : K_COMPACT_SCATTER_SCALAR;
      fp->launches[l].grid[0] = grid;
      ++l;
    }
    pub.n_launches = l;
  } else if (an.tmpl == DISC_TEMPLATE_LOOP) {
    if (sv.rows == 0 || sv.inner == 0) return DISC_OK;
    int want_vec = -1, want_i64 = -1;
    if (force >= 0) {
      if (force > DISC_V_LOOP_SCALAR_I64)
        return set_err(c, DISC_ERR_INVALID_ARG, "forced version does not belong to a loop-fusion pattern");
      want_vec = force == DISC_V_LOOP_VEC || force == DISC_V_LOOP_VEC_I64;
      want_i64 = force == DISC_V_LOOP_VEC_I64 || force == DISC_V_LOOP_SCALAR_I64;
    }
    static const int names[] = {K_LOOP_VEC, K_LOOP_VEC_I64, K_LOOP_SCALAR, K_LOOP_SCALAR_I64};
    bool vec, i64;
    rc = plan_loop(c, sv.rows, sv.inner, V, want_vec, want_i64, names, K_LOOP_VEC_NT, full_aligned(), sv.alg_bytes >= kNonTemporalMinBytes, fp, &fp->launches[0], &vec, &i64);
    if (rc) return rc;
    pub.variant = vec ? (i64 ? DISC_V_LOOP_VEC_I64 : DISC_V_LOOP_VEC) : (i64 ? DISC_V_LOOP_SCALAR_I64 : DISC_V_LOOP_SCALAR);
    pub.n_launches = 1;
  } else if (an.tmpl == DISC_TEMPLATE_ROW_REDUCE) {
    const int n_col_sums = p.gen.n_col_sums;   // outputs summed over the rows, carried along by the row kernels
    const int n_row_reds = p.gen.n_row_reds;   // per-row values reduced over the rows to one number each
    if (sv.rows == 0 && n_row_reds > 0) return set_err(c, DISC_ERR_EMPTY_REDUCE, "reduction over an axis of size 0");
    if (sv.rows == 0 && n_col_sums > 0 && sv.inner > 0)
      return set_err(c, DISC_ERR_EMPTY_REDUCE, "reduction over an axis of size 0");
    if (sv.rows == 0) return DISC_OK;
    if (sv.inner == 0 && an.n_phases == 0) return DISC_OK;   // (no reduction over the rows' axis: nothing to do)
    if (sv.inner == 0) return set_err(c, DISC_ERR_EMPTY_REDUCE, "reduction over an axis of size 0");
    if (sv.inner >= (1ll << 31) - 4096) return set_err(c, DISC_ERR_SHAPE, "row longer than 2^31 elements");
    bool vec = sv.inner >= V / 2 || V == 1;
    bool stream;
    if (force >= 0) {
      if (force < DISC_V_ROW_REG_VEC || force > DISC_V_ROW_STREAM_SCALAR)
        return set_err(c, DISC_ERR_INVALID_ARG, "forced version does not belong to a row-reduce pattern");
      vec = force == DISC_V_ROW_REG_VEC || force == DISC_V_ROW_STREAM_VEC;
    }
    const int v = vec ? V : 1;
    int64_t spr = (sv.inner + v - 1) / v;
    stream = spr > 1024 * (vec ? 3 : 2);
    if (vec) {
      // Rows that write nothing per element: there is no store for the register-resident versions to
      // overlap with the next row's loads, and the streaming version keeps more rows on a CU.  bf16 log-sum-exp,
      // register-resident / streaming, 2^27 elements: 8192 columns 82.0 us / 48.8, 12288 61.4 / 55, 16000 99.1 / 45.
      // Rows of up to 768 slots (blocks of at most 256 threads in the register-resident versions): with enough of
      // them and more than three slots for every lane of a wavefront, where they start on dword boundaries and a lane
      // holds eight slots (two operands: 16384 rows of 2000, 22.6 / 24.9; 2500, 27.3 / 34.6).
      // 16384 rows of 6000 columns 41.1 / 39.7, 4096 33.9 / 28.5, 3000 26.4 / 23.2, 2500 22.2 / 20.4, 2000 20.8 / 17.7;
      // but 1501 15.3 / 16.7, 1024 13.3 / 13.9; odd rows, whose slots the others shift: 4095 34.3 / 35.9, 2049 21.8 /
      // 21.8; 8192 rows of 2500 14.8 / 13.9, 6000 of 4096 17.4 / 14.8, 5000 of 3000 12.2 / 11.7, 4000 of 2500 10.1 / 10.4.
      // Launches beyond the memory-side cache that three slots a lane of 256 lanes fit are bound by the memory, and no faster: 30000
      // rows of 6080 66.0 / 69.6, of 5120 59.9 / 60.9 (16000 rows of 5000 39.1 / 33.6); and of 128 lanes, four-byte elements, from
      // 144 MiB: fp32 sums, 40000 rows of 1240 31.8 / 33.3, of 1400 35.7 / 37.4.
      if (p.gen.row_held) {
        bool dwords = true;
        for (const Access& a : an.accesses)
          if (a.kind == ACC_FULL && (sv.inner * dtype_bytes(a.dtype)) % 4 != 0) dwords = false;
        const bool one = p.gen.stream_held > kStreamHeldSlots;
        const bool three = V <= 4 && spr > 256 && spr <= 384 ? sv.alg_bytes >= (144ll << 20) : spr > 512 && sv.alg_bytes >= (256ll << 20);
        if (spr > 3 * 256 || (force < 0 && one && spr > 3 * 64 && dwords && !three && sv.rows > 16ll * c->n_cus)) stream = true;
      }
      // Sums over the rows and three slots per lane do not fit the registers of a wide block
      // (LayerNorm backward of 24000 columns: 1007 us, 514 in the streaming version)
      if (n_col_sums > 0 && spr > 2 * 1024) stream = true;
    }
    if (force == DISC_V_ROW_STREAM_VEC || force == DISC_V_ROW_STREAM_SCALAR) stream = true;
    else if (force >= 0 && stream) return set_err(c, DISC_ERR_INVALID_ARG, "row too long for the forced register-resident version");
    pub.vec_width = v;
    pub.index_bits = 64;
    fp->spr = spr;
    fp->nslots = 0;
    LaunchRec& L = fp->launches[0];
    L.block = 256;
    // Workspace that covers the launch whatever the alignment of the operands, which a caller does not show
    // when it asks for the size: rows of partial sums, and blocks of the row kernel.
    // (Rows are counted in fp32; own_rows: those of this launch.)
    int64_t most_rows = 0, most_blocks = 0, own_rows = 0;
    // Lanes along the columns, version by column tiles: 64, so that four rows of a block meet in LDS and
    // leave one row of partial sums (GELU backward, 64 / 128 / 256 lanes: 3000 x 2048 12.1 / 12.5 / 13.8 us, 900 x
    // 12000 18.2 / 18.4 / 19.5, 8192 x 16384 136 / 140 / 138, 65536 x 1024 70.1 / 71.7 / 71.7 (two more barriers a block than now), 10000 x 12288 126 / 126
    // / 131; the other way round 16000 x 8192 139 / 135 / 135, 20000 x 1400 38.9 / 36.4 / 37.6).  Large launches of ragged rows run faster with
    // 256 (60000 x 1100 94.7 / 99.3 / 91.2, 12000 x 5001 96.8 / 95.3 / 92.0).
    // (so do rows of more tiles than a grid is high).  Down to one lane for rows of one slot: with eight
    // lanes at least, seven of them idle there (2^24 rows of 8: 786 us / 139; 2^21 of 16: 84.6 / 38.4, of 24: 86.3 /
    // 55.7, of 32: 88.8 / 70.5).
    const int most_tx = (sv.inner % v == 0 || sv.alg_bytes < kNonTemporalMinBytes) && spr <= 64 * 65535ll ? 64 : 256;
    int TX = 1;
    while (TX < most_tx && TX < spr) TX *= 2;
    const int64_t col_tiles = (spr + TX - 1) / TX;
    if (p.gen.row_cols_ok && vec && (force < 0 || force == DISC_V_ROW_REG_VEC) && col_tiles <= 65535) {
      const bool nt = v > 1 && sv.inner % v == 0 && c->row_nt != 0 &&
                      (c->row_nt > 0 || (sv.alg_bytes >= kNonTemporalMinBytes && full_aligned()));
      pub.variant = DISC_V_ROW_REG_VEC;
      L.kid = nt ? K_ROW_COLS_VEC_NT : K_ROW_COLS_VEC;
      // Two blocks per CU with non-temporal accesses, three with plain ones: the chip holds seven, but
      // with more streams in flight the memory delivers less.  Measured (bf16, 2^26 elements; 2 / 3 /
      // 4 / 7 blocks per CU): 4096 columns 71.0 / 73.9 / 77.5 / 79.9 us, 1024 columns 71.1 / 74.3 /
      // 79.9 / 84.4; plain accesses, 1100 columns 104 / 90 / 95 / 108, 5001 columns 102 / 100 / 112 /
      // 104.  Every block writes (and the second launch reads) a row of partial sums: three per
      // CU need eight rows a lane (3000 x 2048, 2.9 / 2 per CU: 16.5 / 13.9 us), and a lane has two rows where
      // that leaves a block per CU (256 x 4096, one / two rows a lane: 9.2 / 8.3).  Numbers in between load the
      // CUs unevenly (2000 x 3072, 3 / 2.6 / 2 per CU: 14.2 / 15.4 / 13.3).  No more rows of partial sums
      // than fit the fixed scratch array.
      // The workspace is enough for both versions: a caller asks for it without saying how its operands
      // will be aligned.
      const int64_t row_groups = (sv.rows + 256 / TX - 1) / (256 / TX);
      auto blocks_per_tile = [&](int per_cu) {
        auto at = [&](int n) {
          const int64_t q = (int64_t)c->n_cus * n / col_tiles;
          return q >= 8 ? q : ((int64_t)c->n_cus * n + col_tiles - 1) / col_tiles;
        };
        const int64_t fill = per_cu == 3 && row_groups < 8 * at(3) ? at(2) : at(per_cu);
        int64_t g = std::min(row_groups, std::min(fill, std::max(at(1), (row_groups + 1) / 2)));
        // Rows of partial sums in fp64 where fp32 ones would show: every one of them rounded once is as much
        // again as the rounding of the result when the terms have both signs, and 1 / number of rows of it
        // when they have one sign.  256 of them for 4096 rows and more are no worse than chains of a
        // few fp32 additions each; a single one is the sum itself.
        const int64_t fit = DISC_STATIC_SCRATCH_BYTES / (4ll * n_col_sums * sv.inner);
        const bool wide = sv.rows < 4096 || std::min(g, fit) < 256;
        g = std::max<int64_t>(1, std::min(g, wide ? fit / 2 : fit));
        return std::make_pair(g, wide && g > 1);
      };
      const auto [grid, fp64_rows] = blocks_per_tile(nt ? 2 : 3);
      const auto plain = blocks_per_tile(3);
      most_rows = plain.first * (plain.second ? 2 : 1);
      L.grid[0] = (uint32_t)grid;
      L.grid[1] = (uint32_t)col_tiles;
      fp->aux[0] = grid;        // rows of partial sums
      fp->aux[1] = TX;
      fp->aux[2] = fp64_rows;
      own_rows = grid * (fp64_rows ? 2 : 1);
      pub.lanes_per_row = TX;
      pub.slots_per_lane = 2;   // rows in flight
      pub.reg_slots = 2;
    } else if (stream) {
      pub.variant = vec ? DISC_V_ROW_STREAM_VEC : DISC_V_ROW_STREAM_SCALAR;
      L.kid = vec ? K_ROW_STREAM_VEC : K_ROW_STREAM_SCALAR;
      // the least block whose registers hold the row; rows up to twice of what the largest one holds
      // still run in it, longer ones (which are read again in every phase anyway) in blocks of 256
      const bool held = vec && p.gen.row_held;
      // (a few rows per CU: more threads to a row, four slots a lane instead; us, four / eight: 1000 x 8000 bf16 9.1 / 9.4, fp32
      // variances 272 x 4150 2.8 / 3.0; 769 to 1024 slots while the chip has work for a few rounds, log-sum-exp 1900 x 7200 11.2
      // / 11.9, 4500 x 8160 17.3 / 19.0, 6000 x 8160 22.6 / 23.8; up to 2048, maximum with position 1200 x
      // 16000 9.1 / 9.7; not longer ones, maximum with position 270 x 20800
      // 6.8 / 5.3, though 3 x 31200 of a maximum alone 2.6 / 2.7)
      const bool few = sv.rows <= (spr <= 3 * 256 ? 4ll : spr <= 256 * kStreamHeldSlots ? 28 : spr <= 512 * kStreamHeldSlots ? 5 : 0) * c->n_cus;
      const int64_t per_lane = held && !few ? p.gen.stream_held : kStreamHeldSlots;
      if (vec && spr <= 2 * 1024 * kStreamHeldSlots) {
        if (held && per_lane > kStreamHeldSlots) L.block = 64;
        while (L.block < 512 && L.block * per_lane < spr) L.block *= 2;
        if (L.block * per_lane < spr) L.block = 1024;
      }
      if (held) {
        if (L.block > 512 || few) L.kid = K_ROW_STREAM_VECW;
        // Held slots are read once.  (The line lies above that of the other non-temporal versions: nothing is
        // written, and inputs of up to 85 MB are still found in the memory-side cache when three of them take turns: 700 x
        // 50257 bf16, 70 MB, 21.1 us / 23.4 with the hint; 16384 x 2000 f32, 131 MB, 23.9 / 21.6; larger ones gain 3-10 %,
        // rows off 16-byte boundaries too.)
        fp->aux[2] = c->row_nt != 0 && (c->row_nt > 0 || sv.alg_bytes >= kNonTemporalMinBytes * 3 / 2);
      }
      // (sums over the rows: a row of partial sums per block in the workspace, so fewer blocks, and for
      // rows that a register-resident version could hold no more than that would need)
      const int64_t most = n_col_sums > 0 ? (spr <= 3 * 1024 ? (int64_t)c->n_cus - 1 : (int64_t)c->n_cus * 2)
                           : L.block > 256 ? (int64_t)c->n_cus * resident_blocks(c, p, L.kid, L.block, 0) : max_grid * 2;
      L.grid[0] = (uint32_t)std::min<int64_t>(sv.rows, most);
      fp->aux[0] = L.grid[0];   // rows of partial sums: one per block
      pub.lanes_per_row = (int)L.block;
      pub.slots_per_lane = (int)((spr + L.block - 1) / L.block);
      pub.reg_slots = !vec ? 1 : (int)(held && L.kid == K_ROW_STREAM_VEC ? p.gen.stream_held : kStreamHeldSlots);
    } else {
      // Lanes per row G and slots per lane nv (<= 2): the pair with the least capacity G * nv that
      // holds the row, two slots per lane on a tie.  G is a power of two.  The kernels accept any
      // multiple of 64 above a wavefront, but the finer steps measured slower: 6-wavefront blocks
      // load the four SIMDs of a CU unevenly (-25 %), 12-wavefront blocks (192 x 4 rows, 384 x 2)
      // leave a CU with one resident block (-10 %), and one slot per lane on more lanes loses to two
      // slots on fewer.  Wavefronts that hold no slot of the row skip the arithmetic anyway.
      struct Shape { int G, block; };
      static const Shape shapes[] = {{1, 256},  {2, 256},  {4, 256},   {8, 256},   {16, 256},  {32, 256},
                                     {64, 256}, {128, 256}, {256, 256}, {512, 512}, {1024, 1024}};
      const int max_nv = vec ? 3 : 2;   // three slots: vector versions only
      int G = 1024, nv = 2, block = 1024;
      auto choose = [&](int64_t slots) {
        int64_t best_cap = -1;
        for (const Shape& s : shapes)
          for (int k = max_nv; k >= 1; --k) {
            if (k == 3 && s.block > 256 && n_col_sums > 0) continue;   // (see above: 12288 columns 986 us)
            const int64_t cap = (int64_t)s.G * k;
            if (cap >= slots && (best_cap < 0 || cap < best_cap)) { best_cap = cap; G = s.G; nv = k; block = s.block; }
          }
      };
      // A ragged end (row length not a multiple of the vector width) as single elements: the row
      // then needs lanes for its WHOLE slots only, and the elements behind them go one each to the
      // first lanes of the row -- in the versions for rows of whole slots, when the pattern has
      // them for this case (no sums over the rows), the row has at least as many lanes as a slot
      // has elements, and the block is a wavefront quad.  Otherwise the ragged end is a slot.
      const bool tail_ok = vec && v > 1 && p.gen.row_tail_ok && sv.inner % v != 0 && sv.inner / v >= 1;
      bool tail = false;
      // (blocks above 256 threads have such a version for two slots per lane only)
      auto tail_fits = [&](int64_t slots) { return G >= v && (block <= 256 || (slots + G - 1) / G <= 2); };
      if (tail_ok) {
        choose(sv.inner / v);
        tail = tail_fits(sv.inner / v);
      }
      if (!tail) {
        choose(spr);
        tail = tail_ok && tail_fits(sv.inner / v);   // (the whole slots alone would have fitted fewer lanes than a slot has elements)
      }
      // Ragged rows of 9 to 12 slots would run on four lanes, with a ragged last slot in every group: with
      // enough of them, eight lanes that take the ragged ends as single elements are faster although a
      // third of them is idle.  300007 rows of 73 / 77 / 85 / 93 / 95 in us, on four and on eight lanes: mixed chain
      // 33.2 / 36.6 / 39.9 / 42.7 / 44.5 and 34.1 / 35.3 / 36.9 / 38.6 / 39.0; softmax 24.7 / 26.2 / 30.3 / 32.7 / 34.3
      // and 22.9 / 23.7 / 27.2 / 29.2 / 29.5; LayerNorm 40.5 .. 51.7 and 39.2 .. 44.1; add + RMS norm 53.6 .. 71.6 and 45.5
      // .. 54.0; log-sum-exp and row amax 19.2 .. 20.1, 12.3 .. 13.9 and 19.0 .. 19.7, 10.1 .. 11.4.  Rows of eight
      // whole slots, one to a lane, gain most: 300007 rows of 65 .. 71, mixed chain 29.8 / 24.2, softmax 17.4 / 14.3, LayerNorm 35.9 /
      // 30.7; attention softmax 128 x 16 x 69 x 69 13.4 / 9.4, 16 x 16 x 71 x 71 5.1 / 4.7.  (Rows of 65, which would gain as
      // much, keep the one schedule that they are held to at any number of rows.  3000 or 1200 rows take the time
      // of a launch either way, 4.7 .. 5.0.)
      if (tail_ok && !tail && G == 4 && v == 8 && sv.inner > 8 * v + 1 && sv.rows >= 4ll * c->n_cus) {
        G = 8;
        tail = true;
      }
      // Sums over the rows, three slots a lane: 200 registers, two blocks on a CU.  Two slots on twice the lanes while
      // every other CU has a row group at most (us, three / two: LayerNorm backward 3000 x 130 12.5 / 10.8, 300 x 140 11.8 / 10.5,
      // 64 x 150 11.5 / 9.9; longer rows, 500 x 700 11.8 / 10.6, would double a workspace that is no longer small;
      // with 312 groups 5000 x 350 15.5 / 16.1, 10000 x 150 14.9 / 15.6; 2000 x 1400 14.7 / 16.6), and blocks of 512 threads for rows that fill two thirds of their lanes (300 x 5500 20.0 / 17.5, 10000 x 6140 95.9
      // / 93.5; 2000 x 5000 28.0 / 29.9).  A row group has a row of partial sums: more rows ask for as many as the fewer ones on
      // twice the lanes do, so that a workspace asked for at the most rows serves them all.
      int64_t fewer_rows_blocks = 0;
      bool count_even = false;
      if (n_col_sums > 0 && nv == 3) {
        const int64_t groups = (sv.rows + 256 / G - 1) / (256 / G);
        if (G <= 16 && 2 * groups > c->n_cus) fewer_rows_blocks = c->n_cus;
        count_even = G == 256 && 3 * spr > 2 * 1024;
        if ((G <= 16 && 2 * groups <= c->n_cus) || count_even) {
          G *= 2;
          nv = 2;
          block = std::max(block, G);
        }
      }
      // Blocks of 1024 threads that walk several rows: the two-slot version for wide blocks has no
      // software pipeline, and with one or two such blocks on a CU nothing else covers the loads of
      // the next row.  The three-slot version (which has one) runs the same rows, from eight of them per
      // CU on (2^27 elements in rows of 16000: mixed chain 190 us / 151 with it, LayerNorm 172 / 149;
      // 13000: 209 / 172 and 192 / 164).  Not where the two-slot version takes the ragged ends as
      // single elements with shifted slots (12289: mixed chain 162 / 184; LayerNorm, unshifted, 224 / 200): that is, not where fp32 row
      // vectors are read, but where the copies of two-byte ones do not fit.
      //
      // Row vectors that can be staged in LDS: bytes of one copy of each, or of a copy for every lane group or
      // shift, whichever are fewer; and bytes of a row of the full-size operands and results.
      bool narrow = false, off_dword = false;
      bool slot_bases = true, line_bases = true;   // full-size operands on boundaries of slots, and of 128 bytes
      int64_t row_bytes = 0, stage_pad = 0;      // (the slot of padding that only shifted copies need)
      for (int eb : p.gen.staged_elem_bytes) {
        narrow = narrow || eb < 4;
        stage_pad += V * eb;
      }
      for (const Access& a : an.accesses) {
        if (a.kind != ACC_FULL) continue;
        row_bytes += sv.inner * dtype_bytes(a.dtype);
        if (a.src_value >= 0) continue;
        const void* ptr = a.is_output ? (outputs ? outputs[a.slot] : nullptr) : (inputs ? inputs[a.slot] : nullptr);
        if (reinterpret_cast<uintptr_t>(ptr) % (uintptr_t)(v * dtype_bytes(a.dtype)) != 0) slot_bases = false;
        if (reinterpret_cast<uintptr_t>(ptr) % 128 != 0) line_bases = false;
        if (dtype_bytes(a.dtype) >= 2 && (sv.inner * dtype_bytes(a.dtype)) % 4 != 0) off_dword = true;
      }
      auto stage_bytes = [&](int64_t groups) {
        int64_t bytes = 0;
        for (int eb : p.gen.staged_elem_bytes)
          bytes += std::min<int64_t>(groups, std::min(V, 16 / eb)) * (((sv.inner + 2 * V) * eb + 15) & ~15ll);
        return bytes;
      };
      const int64_t copies = stage_bytes(block / G), one = stage_bytes(1);
      const bool large = c->row_nt > 0 || sv.alg_bytes >= kNonTemporalMinBytes;
      // LDS for the row vectors of shifted rows: wide blocks of large launches take 64 KiB (bf16 rows, two fp32 vectors, 9585 x
      // 7001, 56 KB, from memory / staged 87.3 / 69.7 us); where three blocks share a CU, or a block has few rows, from memory
      // (three vectors 13419 x 5001, 60 KB, 99.4 / 124; 599 x 7001 6.3 / 7.4).  (Right at the limit, LayerNorm of three two-byte
      // vectors, from memory / staged: 8206 x 8178 89.4 / 77.7, 256 x 8177 5.6 / 7.1.)  fp32 vectors of blocks of 1024 threads, one to a CU,
      // pay for it from six rows a block on (mixed chain 1100 / 1366 / 1700 / 2400 x 12289, from memory 22.0 / 25.7 / 29.9 / 40.9, staged 22.0
      // / 25.6 / 29.4 / 39.7; two of fp32 rows, 7001, from memory 23.3 / 28.1 / 32.6 / 44.6, staged 24.2 / 28.4 / 32.5 / 43.1).
      const bool wide_copies = block > 256 && large && (narrow || block < 1024 || sv.rows >= 6ll * c->n_cus);
      auto fits = [&](int64_t bytes, bool shifted) {
        return bytes <= (shifted && wide_copies ? kMaxShiftedStageBytes : kMaxStageBytes + (large ? stage_pad : 0));
      };
      // Two-byte row vectors, whose rows have plain accesses where they are not shifted: launches beyond what the memory-side
      // cache holds of a few of them in turn (rows scaled by their norm and one vector, 64 MiB, 2396 x 7001, unshifted / shifted,
      // 13.3 / 15.8 us), blocks with one lane group, so that one copy serves it, and rows off dword boundaries (LayerNorm
      // with three, 9585 x 7001 84.2 / 79.1); rows on them where the vectors are a small part of what a row takes anyway (2^26 elements
      // of 4098, one / two / three vectors, 78.7 / 82.7 / 83.6 and 73.7 / 85.7 / 90.1; of 7002, one / two, 77.9 / 77.0 and 72.2 / 70.8).
      auto narrow_copies = [&]() {
        return block == G && c->row_nt != 0 && (c->row_nt > 0 || sv.alg_bytes >= kNarrowShiftMinBytes) && c->row_stage && fits(one, true) &&
               (off_dword || (block <= 256 ? 2 * one <= row_bytes : block <= 512 && 10 * one <= 7 * row_bytes));
      };
      const bool shift_stays = !narrow || narrow_copies();
      const bool piped_wide = vec && block == 1024 && n_col_sums == 0 && sv.rows >= 8ll * c->n_cus && !(tail && p.gen.row_shift_ok && shift_stays);
      if (piped_wide) tail = false;
      if (tail) spr = sv.inner / v;
      nv = (int)((spr + G - 1) / G);
      // Vector slots on the 16-byte boundaries of the tensor (the elements of a row in front of the
      // first boundary become single elements too): when the bases of the full-size operands are
      // aligned to a slot, the row has lanes for up to 2 (V - 1) single elements, and the grid can
      // be cut so that a lane group only meets rows of one alignment (see below).
      // Measured (rows of 2047 .. 4104 bf16 elements, plain accesses): rows that start on dword
      // boundaries run as fast unshifted as rows of whole 16-byte slots (5.14-5.20 against 5.15
      // TB/s) and lose 1-6 % when shifted (more single elements); rows that start off a dword
      // boundary (odd lengths of 2-byte elements) run at 4.90 unshifted and 4.95-5.01 shifted.
      // So the shift is for rows that start off dword boundaries only.
      // Large launches, 64 lanes per row and more (128 for rows on dword boundaries): non-temporal accesses,
      // with the slots on boundaries of whole 128-byte lines of the tensor -- of its one-byte operands too,
      // with 256 lanes; of 64 bytes with 64 -- which leaves more single elements, one to a lane.  On
      // 16-byte boundaries alone the hint loses (the lines between two wavefronts' accesses are written
      // in two parts), on whole lines it gains what it gains on aligned rows.  Mixed chain, 2^28 elements,
      // without and with: rows of 5739 272 / 253 us, 2047 272 / 249, 4095 272 / 248, 8191 250 / 237,
      // 1501 261 / 254, 1023 261 / 258, 4098 260 / 251, 5740 263 / 245; with 32 lanes (515) 269 / 289.  2^28
      // elements of other patterns: bf16 softmax 2047 203 / 180, 4100 204 / 177, 777 205 / 202; fp32 softmax 1501 405 / 378,
      // 8191 403 / 366, 601 405 / 407; log-sum-exp (no element outputs) 1501 99.5 / 91.1, 4095 109 / 108; add + RMS norm 4100
      // 425 / 387; row amax 3001 94.0 / 90.9, 1023 90.1 / 91.9.
      const bool may_shift = tail && p.gen.row_shift_ok && G >= 2 * v - 2 && c->row_shift != 0;   // with operands of the right alignment
      struct Shift { bool shift, lines; };
      auto shifted = [&](bool slots, bool whole_lines) {
        if (!may_shift || !slots) return Shift{false, false};
        bool lines = G >= kMinLinesG && c->row_nt != 0 && (c->row_nt > 0 || sv.alg_bytes >= kNonTemporalMinBytes);
        // (a base on a slot but off a line still gains from 128 lanes on, 16 bytes past a line without / with: bf16
        // softmax 2047 76.6 us / 72.2, 5739 77.3 / 71.0, add + RMS norm 4095 159 / 151; with 64 add + RMS norm 777 159 / 168)
        if (!whole_lines && G < kMinLinesEvenG) lines = false;
        // An operand like the mask [B, 1, 1, S] of a softmax has its own boundaries, which shifted slots miss: then
        // only where two slots per lane are nearly full, and in wide blocks (f16, without / with lines: S = 777 170 us /
        // 177, 1501 177 / 180, 1700 159 / 164, 3001 157 / 166, 5742 116 / 123; 2047 143 / 137, 4098 105 / 103, 8191 206 / 194).
        if (p.gen.row_narrow_late && block <= 256 && !(G >= 128 && nv == 2 && 8 * spr >= 7 * 2 * G)) lines = false;
        lines = lines && (off_dword || G >= kMinLinesEvenG);
        bool shift = off_dword || lines;
        // Row vectors.  Shifted slots read copies shifted alike, one for every lane group or shift, and every block writes them.
        // That pays in large launches while they are no more than 3.5 times a row (unshifted / shifted, us: one fp32 vector of bf16 rows in
        // four copies, LayerNorm 44709 x 1501 78.0 / 75.0, mixed chain 44709 x 1501 69.8 / 65.8; two of fp32 rows in two 44709 x 1501 150 / 137;
        // but two of bf16 rows in four copies 32800 x 1023 41.2 / 45.0, three 41.7 / 48.2).  Beyond, and in smaller launches, rows are not
        // shifted (mixed chain 3000 x 1023 5.6 / 6.6).  One copy a block always pays; where it does not fit, fp32 vectors are read
        // from memory (three vectors 11693 x 5739, unshifted / shifted and from memory, 108 / 95.2; two 8207 x 8177 94.4 / 79.0).
        if (shift && one > 0) {
          if (narrow) shift = lines && narrow_copies();   // (from memory their slots are off dword boundaries)
          else if (c->row_stage && block > G && fits(one, false)) shift = large && fits(copies, true) && 2 * copies <= 7 * row_bytes;
        }
        return Shift{shift, lines && shift};
      };
      auto [shift, lines] = shifted(slot_bases, line_bases);
      const bool aligned_shift = shifted(true, true).shift;
      const int align = lines ? std::min(128, G / 2) : v;    // elements
      int inst = piped_wide ? 3 : std::max(nv, 2);   // instantiated slots per lane: 2 or 3
      int kid_aligned = 0, kid_any = 0;     // kernel for aligned operands, and for others
      pub.variant = vec ? DISC_V_ROW_REG_VEC : DISC_V_ROW_REG_SCALAR;
      L.block = (uint32_t)block;
      L.plan_kind = 1;
      L.rp.G = G;
      L.rp.log2G = ilog2_ceil(G);
      L.rp.nv = nv;
      L.rp.rpb = block / G;
      uint32_t lds_unshifted = 0;           // LDS of the same launch with operands off the boundaries of slots
      int kid_unstaged = -1;                // kernel of fewer rows, where they read the row vectors from memory
      {
        // Staged or not, whatever the alignment of the operands: a single-shape module has one kernel for all of them.
        const bool stage = vec && V > 1 && c->row_stage && one > 0 && fits(aligned_shift ? copies : one, aligned_shift);
        L.rp.flags = (stage ? 1 : 0) | (n_col_sums == 0 ? 0 : 2);
        L.dyn_lds = !stage ? 0 : (uint32_t)(shift ? copies : one);
        lds_unshifted = stage ? (uint32_t)one : 0;
        const bool wide_version = block > 256;
        // Non-temporal version (blocks of 256 threads, vector width only).  Host rule, measured on
        // softmax and LayerNorm sweeps: the hint gains 5-15 % when every row starts and ends on a
        // 16-byte boundary (row length a multiple of the vector width, aligned bases) and either
        // every row is a whole number of 128-byte cache lines (from 128 elements on) or the row has
        // at least 512 elements.  Rows whose first and last cache lines are shared with their
        // neighbours lose with it (-25 % for 360- or 464-element rows, -30 % for short odd rows),
        // as do operands that are read more than once, which never get the hint.  Small launches
        // (kNonTemporalMinBytes) keep the plain version: their results may be consumed from cache.
        // rows of whole slots (row length a multiple of the vector width) take the versions without
        // any ragged-tail path: _e, or _nt under the rule above
        const bool even = vec && V > 1 && !wide_version && (sv.inner % V == 0 || tail);
        bool nt = false;
        if (even && !tail && c->row_nt != 0) {
          nt = c->row_nt > 0;
          if (c->row_nt < 0 && sv.inner >= 128 && sv.alg_bytes >= kNonTemporalMinBytes) {
            bool whole_lines = true;
            for (const Access& a : an.accesses)
              if (a.kind == ACC_FULL && (sv.inner * dtype_bytes(a.dtype)) % 128 != 0) whole_lines = false;
            nt = whole_lines || sv.inner >= 512;
          }
        }
        auto version = [&](bool hint) {
          return K_ROW_BASE + row_kernel_index(!vec, inst, wide_version, stage, hint ? 1 : tail ? 3 : even ? 2 : 0);
        };
        kid_aligned = version(nt);
        L.kid = nt && c->row_nt < 0 && !full_aligned() ? version(false) : kid_aligned;
        kid_any = nt && c->row_nt < 0 ? version(false) : kid_aligned;
        if (stage && tail && one > kMaxStageBytes) kid_unstaged = K_ROW_BASE + row_kernel_index(!vec, inst, wide_version, false, 3);
      }
      // grid-stride over row groups: a small whole number of rounds of the blocks the chip holds
      // at once.  Measured: with plenty of rows, blocks of one wavefront-quad do best with three
      // rounds (the hardware does not fill every CU to the computed residency in the first round;
      // later blocks even that out); the wide blocks, and any launch that would leave a block
      // fewer than four row groups, with one (each new block pays an unpipelined first row and
      // the staging of the row vectors)
      const int rpb = (int)L.block / G;
      const int64_t ngroups = (sv.rows + rpb - 1) / rpb;
      // Sums over the rows of 1025 .. 1536 slots: blocks of 1024 threads, half as many as there would be of 512
      // (three slots per lane), so two rounds of them: a lane's chain of fp32 additions stays as short (relative
      // rms error of dgamma, LayerNorm backward 32768 x 9000, one round / two: 2.1e-7 / 1.55e-7; 436
      // us / 450, most of it the second row of partial sums per CU).  Not where that does not fit ws_limit.
      bool two_rounds = n_col_sums > 0 && vec && block == 1024 && spr <= 3 * 512;
      {
        int64_t cells, bytes;
        if (mul_ovf(2ll * c->n_cus, sv.inner, &cells) || mul_ovf(cells, 4ll * n_col_sums, &bytes) ||
            (uint64_t)bytes + 8ull * (uint64_t)n_row_reds * (uint64_t)c->n_cus + 256 > ws_limit)
          two_rounds = false;
      }
      auto blocks_with = [&](int kid, uint32_t lds) {
        int64_t per_cu = resident_blocks(c, p, kid, L.block, lds);
        // Ragged rows with staged vectors: at most 24 wavefronts on a CU (whole blocks: six of 256 threads, three of 512, one of
        // 1024).  With more the memory delivers less in launches of one round (us, 32 / 28 / 24: fp32 LayerNorm of one vector 21592 x 777
        // 43.4 / 37.1 / 36.9, 40427 x 415 44.7 / 40.8 / 39.5; 28 / 24, of two 21592 x 777 46.6 / 38.4, 65280 x 257 49.9 / 43.6, 8196 x 2047
        // 44.3 / 39.4); several rounds take it either way (of two 86369 x 777 142.7 / 139.2, 130308 x 515 152.9 / 156.2; fp32 rows
        // scaled by their norm 65154 x 515 52.8 / 54.5).
        if (tail && lds > 0) per_cu = std::min<int64_t>(per_cu, std::max<int64_t>(1, 24 * 64 / L.block));
        const int64_t held = (int64_t)c->n_cus * per_cu;
        // (with sums over the rows every block writes a row of partial sums: one round, or two)
        const int rounds = c->row_rounds > 0 ? c->row_rounds
                           : (L.block > 256 || n_col_sums > 0 ? (two_rounds ? 2 : 1) : (int)std::max<int64_t>(1, std::min<int64_t>(3, ngroups / (held * 4))));
        return std::min<int64_t>(ngroups, held * rounds);
      };
      auto blocks_of = [&](int kid) { return blocks_with(kid, L.dyn_lds); };
      auto odd = [&](int64_t g) { return g > 2 && g % 2 == 0 && g < ngroups ? g - 1 : g; };
      int64_t grid = blocks_of(L.kid);
      for (const int kid : {kid_aligned, kid_any})
        if (n_col_sums + n_row_reds > 0) most_blocks = std::max(most_blocks, may_shift || count_even ? blocks_of(kid) : odd(blocks_of(kid)));
      // (a caller that asked with aligned operands, or with none, launches with others: unshifted, less LDS)
      if (may_shift && n_row_reds > 0) most_blocks = std::max(most_blocks, blocks_with(kid_any, lds_unshifted));
      if (kid_unstaged >= 0 && n_row_reds > 0) most_blocks = std::max(most_blocks, blocks_with(kid_unstaged, 0));
      most_blocks = std::max(most_blocks, fewer_rows_blocks);
      // An odd grid: with an even one a block of one row per iteration would only ever see even or
      // only odd rows, and when the row length is odd every other row starts two bytes off a
      // dword -- half of the blocks would run ~20 % slower all the time and set the kernel's time
      // (measured: +14-18 % on 4095- and 5739-wide rows).  With an odd grid every block walks
      // through all alignments of its rows, whatever the rows per block.
      if (shift) {
        // rows of one alignment per lane group: (distance between its rows) x (row length) must be a
        // multiple of the vector width
        int64_t m = align / std::gcd<int64_t>(sv.inner % align, align);
        m /= std::gcd<int64_t>(m, rpb);
        if (grid >= m) grid -= grid % m;
        else shift = false;
      }
      if (shift) L.rp.flags |= 4 | align << 8 | (lines ? 8 : 0);
      else grid = odd(grid);
      L.grid[0] = (uint32_t)grid;
      // rows of partial sums: one per block of 256 threads, one per lane group of a wider block
      const int64_t per_block = L.block <= 256 ? 1 : (int64_t)L.block / std::max(G, 64);
      fp->aux[0] = grid * per_block;
      most_rows = most_blocks * per_block;
      pub.lanes_per_row = G;
      pub.slots_per_lane = nv;
      pub.reg_slots = inst;
    }
    pub.n_launches = 1;
    if (n_col_sums == 0) fp->aux[0] = 0;
    if (n_row_reds > 0) fp->aux[1] = L.grid[0];
    own_rows = std::max(own_rows, fp->aux[0]);
    most_rows = std::max(most_rows, own_rows);
    most_blocks = std::max<int64_t>(most_blocks, L.grid[0]);
    // workspace: n_col_sums planes of [partial rows, inner] (fp32, or fp64 from the version by column
    // tiles), which the second launch adds up; behind them one partial result per block and reduction
    // of per-row values, folded by a last launch of one block
    auto layout = [&](int64_t partial_rows, int64_t blocks, size_t* reds_at, size_t* total) {
      int64_t cells, bytes = 0;
      if (n_col_sums > 0 && (mul_ovf(partial_rows, sv.inner, &cells) || mul_ovf(cells, 4ll * n_col_sums, &bytes))) return false;
      *reds_at = ((size_t)bytes + 255) / 256 * 256;
      *total = n_row_reds > 0 ? *reds_at + (size_t)n_row_reds * (size_t)blocks * 4 : (size_t)bytes;
      return true;
    };
    size_t unused;
    if (!layout(own_rows, L.grid[0], &fp->ws_off[1], &fp->ws_need) || !layout(most_rows, most_blocks, &unused, &pub.workspace_bytes))
      return set_err(c, DISC_ERR_SHAPE, "workspace size overflows int64");
    if (n_col_sums > 0) {
      fp->ws_off[0] = 0;
      LaunchRec& L1 = fp->launches[1];
      L1.kid = K_COLSUM_FINISH;
      L1.block = 256;
      L1.grid[0] = (uint32_t)std::min<int64_t>((sv.inner + 15) / 16, max_grid * 4);   // 16 columns per block
      pub.n_launches = 2;
    }
    if (n_row_reds > 0) {
      LaunchRec& Lr = fp->launches[pub.n_launches++];
      Lr.kid = K_ROWRED_FINISH;
      Lr.block = 1024;
      Lr.grid[0] = 1;
    }
  } else {
    // column reduce: canonical [outer, mid, inner], rows = outer * mid
    const int64_t outer = an.mid_group == 1 ? sv.group[0] : 1;
    const int64_t mid = sv.mid, inner = sv.inner;
    if (outer == 0 || inner == 0) return DISC_OK;
    if (mid == 0) return set_err(c, DISC_ERR_EMPTY_REDUCE, "reduction over an axis of size 0");
    if (mid >= (1ll << 31) - 1) return set_err(c, DISC_ERR_SHAPE, "reduced axis longer than 2^31");
    // the column tiles are the x dimension of the grids (no grid stride across columns)
    if (inner >= (1ll << 31) - 4096) return set_err(c, DISC_ERR_SHAPE, "column reduce: more than 2^31 columns");
    constexpr int64_t kTwoLaunchChunks = 32;
    int want_vec = -1, want_strip = -1, want_two = -1;
    if (force >= 0) {
      const bool two = force == DISC_V_COL_2STAGE_VEC || force == DISC_V_COL_2STAGE_SCALAR;
      if ((force < DISC_V_COL_3STAGE_VEC || force > DISC_V_COL_STRIP_SCALAR) && !two)
        return set_err(c, DISC_ERR_INVALID_ARG, "forced version does not belong to a column-reduce pattern");
      if (two && !p.gen.has_epilogue)
        return set_err(c, DISC_ERR_INVALID_ARG, "the two-launch version needs an output that keeps the reduced axis");
      want_vec = force == DISC_V_COL_3STAGE_VEC || force == DISC_V_COL_STRIP_VEC || force == DISC_V_COL_2STAGE_VEC;
      want_strip = force == DISC_V_COL_STRIP_VEC || force == DISC_V_COL_STRIP_SCALAR;
      want_two = two;
    }
    bool vec;
    {
      const int64_t spr_v = (inner + V - 1) / V;
      vec = 1.0 - (double)inner / (double)(spr_v * V) <= 0.25;
      if (want_vec >= 0) vec = want_vec != 0;
    }
    const int v = vec ? V : 1;
    const int64_t spr = (inner + v - 1) / v;
    // Small problems: one launch, a block per strip of columns (reduce, finish and epilogue in the
    // same kernel), up to about a million elements.
    int64_t total;
    const bool million = !mul_ovf(outer * mid, inner, &total) && total <= (1ll << 20);
    // strips of >= 32 bytes per row keep the accesses coalesced; narrower strips = more blocks
    int strip_gc = 1;
    while (strip_gc < 64 && (strip_gc * (vec ? 16 : 4) < 32 || spr / (strip_gc * 2) >= 64)) strip_gc *= 2;
    strip_gc = std::min<int>(strip_gc, 1 << ilog2_ceil(std::min<int64_t>(spr, 64)));
    const int64_t lane_rows = mid / (256 / strip_gc);       // rows that a lane walks, twice
    // A strip that the block can hold in registers is read once (col_held): few rows leave room for more and narrower
    // strips, one for every CU, many rows take more threads, four to eight rows to a lane (64 strips / 256: 256 x 4096 7.7 us
    // / 5.4, 100 x 4096 5.3 / 4.8; 700 x 1024 6.0 / 6.8, 500 x 2000 6.4 / 7.5; 207 / 413: 159 x 3300 4.5 / 5.5; 256 / 512 /
    // 1024 threads: 300 x 1024 5.0 / 4.8 / 5.7,
    // 700 x 1024 - / 6.0 / 6.4, 1000 x 1024 - / 7.6 / 7.3).  With a batch there are strips enough, and rows fewer than half
    // of a block's lanes down the rows leave these idle: 64 strips an entry and wider ones (maximum with position 10 x
    // 34 x 1816 16.9 / 9.3, sum 7 x 4 x 10332 6.5 / 2.8).  Maxima with positions are too dear to merge over 16 wavefronts
    // (2 x 1677 x 72 13.4 with 1024 threads, 10.9 in two passes, 9.2 with 512), and for a second round of blocks (held / two
    // passes: 130 x 133 x 45, 780 blocks, 10.5 / 11.2; 175 x 133 x 45, 1050, 14.6 / 12.7; 10 x 34 x 1816, 1140, 9.3 / 8.2).
    uint32_t strip_block = 256;
    bool in_regs = false;
    if (vec && p.gen.col_held) {
      const bool narrow = mid <= 256 && outer < 4;
      int g = 1;
      auto strips = [&]() { return (spr + g - 1) / g; };
      while (g < 64 && (g * 16 < 32 || (narrow ? strips() > 256 / outer : spr / (g * 2) >= 64) || (strips() * outer > c->n_cus && 256 / (g * 2) >= mid)))
        g *= 2;
      g = std::min<int>(g, 1 << ilog2_ceil(std::min<int64_t>(spr, 64)));
      if (mid > (int64_t)kColHeldRows * (256 / g)) g = std::min(g, 16);     // (all that a block above 256 threads takes)
      uint32_t b = 256;
      if (g <= 16 && mid > 4 * (256 / g)) b = 512;
      if (g <= 16 && mid > 6 * (512 / g) && !p.gen.col_argmax) b = 1024;
      const bool resident = strips() * outer * b <= (int64_t)c->n_cus * 1024;
      if (mid <= (int64_t)kColHeldRows * (b / g) && (resident || !p.gen.col_argmax)) {
        strip_gc = g;
        strip_block = b;
        in_regs = true;
      }
    }
    // Many rows to a lane: two launches then, if the caller's workspace allows them.  What counts is the rows that a
    // lane of the two passes walks, whatever the length of the axis; one launch / two, us, single elements: 26 rows (6
    // x 3300 x 2) 4.9 / 7.0, 43 (11000 x 1) 6.1 / 7.0, 49 (12623 x 1) 6.5 / 7.0, 47 (1500 x 5) 6.6 / 6.2, 64 (2040 x 5) 7.8 / 6.2, 344 (11000 x 5) 32.7 /
    // 7.3; slots: 12 (1500 x 40) 8.7 / 9.9, 16 (4100 x 8) 8.6 / 9.5, 20 (2600 x 40) 10.4 / 10.0, 32 (4100 x 40) 15.1 / 10.8.
    // Held strips: 10 (1300 x 777) 9.3 / 10.4, 16 (2040 x 20) 6.3 / 7.8, (6 x 2040 x 64) 8.7 / 9.0, but from 2 MB of operand on
    // the pieces of a row meet in the caches of too few CUs (2040 x 512 10.6 / 8.4, 2600 x 256 11.3 / 7.8), unless a strip
    // is whole rows (40 x 2600 x 8 6.9 / 8.5, 3300 x 8 6.7 / 7.7).
    const bool few_bytes = sv.alg_bytes <= (4ll << 20);
    const bool long_axis = p.gen.has_epilogue && mid > 1024 &&
                           (in_regs ? spr > strip_gc && (lane_rows > 20 || (lane_rows > 12 && !few_bytes)) : lane_rows > (!vec ? 52 : p.gen.col_argmax ? 24 : 20));
    const bool small = million && !long_axis;
    auto plan_strip = [&]() {
      const int GC = strip_gc;
      const int64_t col_tiles = (spr + GC - 1) / GC;
      DeviceColPlan cp{GC, ilog2_ceil(GC), 1, 0, mid, outer, 0};
      fp->aux[0] = 0;
      fp->aux[1] = outer * inner * 8;
      fp->ws_off[0] = 0;
      fp->ws_off[1] = 0;
      // (with an epilogue the reduce results stay in registers; without, they go to the planes)
      pub.workspace_bytes = p.gen.has_epilogue ? 0 : (size_t)p.gen.n_red_planes * (size_t)fp->aux[1];
      pub.variant = vec ? DISC_V_COL_STRIP_VEC : DISC_V_COL_STRIP_SCALAR;
      pub.lanes_per_row = GC;
      pub.vec_width = v;
      pub.index_bits = 64;
      LaunchRec& L0 = fp->launches[0];
      L0.kid = !vec ? K_COL_STRIP_SCALAR : p.gen.col_held && !in_regs ? K_COL_STRIP_VECL : K_COL_STRIP_VEC;
      L0.block = strip_block;
      L0.grid[0] = (uint32_t)col_tiles;
      L0.grid[1] = (uint32_t)std::min<int64_t>(outer, 65535);
      L0.plan_kind = 2;
      L0.cp = cp;
      pub.n_launches = 1;
      for (int k2 = 0; k2 < 3; ++k2) pub.grid[0][k2] = L0.grid[k2];
      pub.block[0][0] = L0.block;
      pub.block[0][1] = pub.block[0][2] = 1;
      pub.lds_bytes[0] = 0;
      snprintf(pub.kernel[0], sizeof pub.kernel[0], "%s%s", p.gen.prefix.c_str(), kernel_name(L0.kid));
      return DISC_OK;
    };
    if (want_strip >= 0 ? want_strip != 0 : small) return plan_strip();
    // Lanes along the columns per block: 16 lanes of one vector each (256 bytes of a row: two
    // whole cache lines) unless the rows are narrower; the other lanes of the block run down the
    // rows.  Narrow column tiles give the grid its width: with 64 lanes across, 1024 fp32 columns
    // are only 4 tiles, and the chunks of the reduced axis would have to supply all the parallelism.
    // (narrow tensors: 8 or 4 lanes across when that yields more blocks, down to 64-byte row pieces)
    int GC = 1 << ilog2_ceil(std::min<int64_t>(spr, 16));
    {
      auto blocks_at = [&](int gc) {
        const int64_t t = (spr + gc - 1) / gc * std::min<int64_t>(outer, 65535);
        const int64_t maxc = std::max<int64_t>(1, mid / (4ll * (256 / gc)));
        return std::min<int64_t>(t * std::min<int64_t>(kTwoLaunchChunks, maxc), (int64_t)c->n_cus * 2);
      };
      int best = GC;
      for (int gc = GC >> 1; gc >= 4; gc >>= 1)
        if (blocks_at(gc) > blocks_at(best)) best = gc;
      GC = best;
    }
    const int TY = 256 / GC;
    const int64_t col_tiles = (spr + GC - 1) / GC;
    const int64_t tiles = col_tiles * std::min<int64_t>(outer, 65535);
    // Chunks of the reduced axis: enough blocks for two per CU, at least four rows per row-lane.
    // Up to kTwoLaunchChunks chunks the second launch can afford to merge the partials of its own
    // columns in every block (a few loads per lane), which saves the finish launch and the round
    // trip of the reduce results through memory: the two-launch version.  A reduced axis so long
    // and narrow that it needs more chunks than that keeps the separate finish launch.
    const int64_t max_chunks = std::max<int64_t>(1, mid / (4ll * TY));
    int64_t nchunk = ((int64_t)c->n_cus * 2 + tiles - 1) / tiles;
    nchunk = std::max<int64_t>(1, std::min<int64_t>(nchunk, max_chunks));
    bool two = p.gen.has_epilogue && (nchunk <= kTwoLaunchChunks || million);
    if (want_two >= 0) two = want_two != 0;
    if (two) nchunk = std::min<int64_t>(nchunk, kTwoLaunchChunks);
    else nchunk = std::min<int64_t>(std::max<int64_t>(1, std::min<int64_t>(((int64_t)c->n_cus * 4 + tiles - 1) / tiles, max_chunks)), 1024);
    const int64_t chunk_rows = (mid + nchunk - 1) / nchunk;
    nchunk = (mid + chunk_rows - 1) / chunk_rows;
    // pieces of a row that a block takes: whole 128-byte lines?
    bool lines = true;
    int64_t row_bytes = 0;
    for (const Access& a : an.accesses) {
      if (a.kind != ACC_FULL || a.is_output) continue;
      if (inner * dtype_bytes(a.dtype) % 128 != 0 || (int64_t)GC * v * dtype_bytes(a.dtype) < 128) lines = false;
      row_bytes = std::max(row_bytes, inner * dtype_bytes(a.dtype));
    }
    // (fewer than 2^31 blocks in either launch)
    const bool lists = !lines && col_tiles < (1 << 15);
    DeviceColPlan cp{GC, ilog2_ceil(GC), (int32_t)nchunk, lists, chunk_rows, outer, 0};
    int64_t cells, red_bytes;
    if (mul_ovf(outer * nchunk, inner, &cells) || mul_ovf(cells, (int64_t)p.gen.n_acc_cells * 8, &red_bytes))
      return set_err(c, DISC_ERR_SHAPE, "workspace size overflows int64");
    // (no workspace for a problem that fits one launch: one launch.  So do single-shape modules, which hold one
    // plan for callers with and without a workspace.)
    if (million && long_axis && force < 0 && (p.is_static || (uint64_t)red_bytes > ws_limit)) return plan_strip();
    fp->aux[0] = cells;                 // cells per accumulator-field plane
    fp->aux[1] = outer * inner * 8;     // bytes per reduce-result plane
    fp->ws_off[0] = 0;
    fp->ws_off[1] = ((size_t)red_bytes + 255) / 256 * 256;
    pub.lanes_per_row = GC;
    LaunchRec& L0 = fp->launches[0];
    L0.kid = vec ? K_COL_PARTIAL_VEC : K_COL_PARTIAL_SCALAR;
    L0.grid[0] = (uint32_t)col_tiles;
    L0.grid[1] = (uint32_t)nchunk;
    L0.grid[2] = (uint32_t)std::min<int64_t>(outer, 65535);
    L0.plan_kind = 2;
    if (two) {
      // second launch: column tiles x row ranges, about eight blocks per CU; every lane gets at
      // least four rows so that the merge of the partials stays a small part of the block's work
      int64_t row_blocks = std::max<int64_t>(1, ((int64_t)c->n_cus * 8 + tiles - 1) / tiles);
      row_blocks = std::min<int64_t>(std::min<int64_t>(row_blocks, max_chunks), 65535);
      cp.epi_rows = (mid + row_blocks - 1) / row_blocks;
      row_blocks = (mid + cp.epi_rows - 1) / cp.epi_rows;
      pub.workspace_bytes = (size_t)red_bytes;   // partials only: the reduce results stay in registers
      pub.variant = vec ? DISC_V_COL_2STAGE_VEC : DISC_V_COL_2STAGE_SCALAR;
      pub.vec_width = v;
      pub.index_bits = 64;
      L0.cp = cp;
      LaunchRec& L1 = fp->launches[1];
      // non-temporal stores for large launches with aligned rows: the results then do not push the
      // operand, which the second launch reads again, out of the memory-side cache
      const bool nt = vec && v > 1 && inner % v == 0 && c->row_nt != 0 &&
                      (c->row_nt > 0 || (sv.alg_bytes >= kNonTemporalMinBytes && full_aligned()));
      // This is the last read of the operands, and the hint on the loads as well gains where the row pieces of
      // a block are whole 128-byte lines, i.e. nobody else wants the rest of a line (fp32, stores only / both: 60000 x
      // 512 66.3 / 61.0 us, 40000 x 768 73.6 / 65.4, 20000 x 2016 88.9 / 77.8, 65536 x 1024 130.9 / 128.9); with
      // pieces of 64 bytes, or rows that end inside a line, it loses (60000 x 256 52.8 / 62.5, 90000 x 384 116 / 130;
      // 30000 x 1000 80.8 / 91.6, 7857 x 3628 84.3 / 93.2, 276620 x 248 306 / 373, all without lists).
      // Without whole lines the blocks come in lists, whose neighbours write the parts of a line shortly after
      // one another: up to 224 MiB, for rows of 3840 bytes and more and for rows of whole lines in smaller pieces the hint on the stores still gains, beyond it the plain
      // store does (stores with the hint / plain: 30000 x 700 56.8 / 60.8, 40000 x 700 78.9 / 80.9, 50000 x 700 113.6 / 102.2, 65536 x
      // 500 98.5 / 86.5, 65536 x 900 184 / 177, 65536 x 1000 149 / 177, 40000 x 1500 158 / 171, 20000 x 3000 133 / 159).  With one
      // operand rows of 3840 bytes are where a block's pieces become 256 bytes wide; batches have such pieces of shorter rows, and keep the plain
      // store (3 x 20000 x 500 71.0 / 61.6, 8 x 6000 x 700 77.9 / 70.4; but 40 x 2000 x 700 133 / 141), as two operands of 2 and 4 bytes have narrower ones
      // of longer rows, and the hint (30000 x 1000 86.5 / 92.0, 65536 x 1000 233 / 227).
      const bool nts = nt && (sv.alg_bytes < (224ll << 20) || row_bytes >= 3840 || row_bytes % 128 == 0);
      L1.kid = !vec ? K_COL_EPI2_SCALAR : nt && (lines || c->row_nt > 0) ? K_COL_EPI2_VEC_NT : nts ? K_COL_EPI2_VEC_NTS : K_COL_EPI2_VEC;
      L1.grid[0] = (uint32_t)col_tiles;
      L1.grid[1] = (uint32_t)row_blocks;
      L1.grid[2] = (uint32_t)std::min<int64_t>(outer, 65535);
      L1.plan_kind = 2;
      L1.cp = cp;
      pub.n_launches = 2;
    } else {
      pub.workspace_bytes = fp->ws_off[1] + (size_t)p.gen.n_red_planes * (size_t)fp->aux[1];
      pub.variant = vec ? DISC_V_COL_3STAGE_VEC : DISC_V_COL_3STAGE_SCALAR;
      L0.cp = cp;
      LaunchRec& L1 = fp->launches[1];
      L1.kid = K_COL_FINISH;
      L1.grid[0] = (uint32_t)((inner + 15) / 16);   // 16 columns per block
      L1.grid[1] = (uint32_t)std::min<int64_t>(outer, 65535);
      L1.plan_kind = 2;
      L1.cp = cp;
      pub.n_launches = 2;
      if (p.gen.has_epilogue) {
        static const int names[] = {K_COL_EPI_VEC, K_COL_EPI_VEC_I64, K_COL_EPI_SCALAR, K_COL_EPI_SCALAR_I64};
        bool v2, i64;
        rc = plan_loop(c, sv.rows, inner, V, vec ? 1 : 0, -1, names, K_COL_EPI_VEC_NT, full_aligned(), sv.alg_bytes >= kNonTemporalMinBytes, fp, &fp->launches[2], &v2, &i64);
        if (rc) return rc;
        pub.n_launches = 3;
      } else {
        pub.vec_width = v;
        pub.index_bits = 64;
      }
    }
  }
  for (int l = 0; l < pub.n_launches; ++l) {
    for (int k = 0; k < 3; ++k) pub.grid[l][k] = fp->launches[l].grid[k];
    pub.block[l][0] = fp->launches[l].block;
    pub.block[l][1] = pub.block[l][2] = 1;
    pub.lds_bytes[l] = fp->launches[l].dyn_lds;
    snprintf(pub.kernel[l], sizeof pub.kernel[l], "%s%s", p.gen.prefix.c_str(), kernel_name(fp->launches[l].kid));
  }
  return DISC_OK;
}

// The workspace limit of a plan that does with as little as the pattern can (column reduces: none where the strip
// version runs; what the others need does not depend on a limit that a caller's workspace sets).
size_t least_limit(const Pattern& p) { return p.an.tmpl == DISC_TEMPLATE_COL_REDUCE ? 0 : SIZE_MAX; }

// A row reduce with a transposed operand in one kernel: batch x per rows of `inner` elements.  false: two kernels.
bool plan_xpose(const disc_ctx* c, int64_t per, int64_t batch, int64_t inner, int V, FullPlan* fp) {
  // Strips of 8 rows (16 bytes of an operand row) in 512 threads; of 16 where that still leaves strips for the chip --
  // fewer accesses to a cache line -- on 32 lanes a row, or 64 in 1024 threads for long rows; of 32 where there are
  // thousands.  bf16 softmax, strips of 8 / 16 / 32, us: 1500 x 5000 (of the operand) 11.9 / 13.2 / 14.8, 2500 x 5000 17.6 /
  // 18.6 / 22.1, 300 x 8192 6.2 / 5.7 / 5.6, 3000 x 8000 37.4 / 26.5 / -, 200 x 200000 76 / 45.5 / 38.1, 1000 x 60000 77 / 62 / 59.
  // Against two kernels: 2000 x 100 5.4 / 8.0, 1000 x 8000 9.5 / 15.1, 2000 x 4000 11.4 / 15.5, 3000 x 2001 11.5 / 15.5, 3500 x 5000
  // 23.0 / 28.9, 8192 x 8192 95.4 / 107.  Rows beyond 4096 elements leave one strip to a CU, whose load, arithmetic and
  // stores follow one another, 20 us however many there are: with several strips for every CU, or one for most or all of
  // them (6000 x 2200 24.3 / 20.5, 4500 x 2600 21.0 / 20.0, 6000 x 3000 24.7 / 28.1, 4500 x 4000 20.9 / 29.3, 8192 x 4000 38.8 / 50.4, 6000 x
  // 4090 26.0 / 38.9, 6000 x 4096 29.6 / 38.6, 8192 x 4096 38.8 / 43.9, 6000 x 4097, a second round for one strip, 45.4 / 38.0; 8192 x 64 14.6 / 10.1, 5000 x 6200 45.3 / 47.5, 6000 x 7000 55.8 / 65.1).  (4000 x 300
  // 9.7 / 9.2 and 4000 x 800 12.0 / 11.0 are on the wrong side of the line; 3200 x 500 8.5 / 9.7, 3600 x 1000 11.4 / 11.8.)
  const int64_t strips16 = (per + 15) / 16 * batch;
  if (inner > 64 * V * 8 && strips16 < c->n_cus * 3 / 2 && !(strips16 > c->n_cus * 2 / 3 && strips16 <= c->n_cus)) return false;
  int G = 64, B = 512, nv = 0;
  if (strips16 >= 8ll * c->n_cus && inner <= 16 * V * 12 && per >= 32) G = 16;
  else if (strips16 >= c->n_cus * 7 / 4 || inner > 64 * V * 8) {
    if (inner <= 32 * V * 12) G = 32;
    else B = 1024;
  }
  for (int k : kXposeSlots)
    if (nv == 0 && (int64_t)G * V * k >= inner) nv = k;
  const int rpb = B / G;
  if (nv == 0 || per < rpb || per > (1 << 18)) return false;
  const int64_t strips = (per + rpb - 1) / rpb, blocks = (strips * batch + 7) / 8 * 8;
  // (a launch has less than 2^32 threads)
  if (blocks * B >= (1ll << 32)) return false;
  // Operand rows of an odd number of two-byte elements: every access is off dword boundaries, which shows where a few strips walk
  // many rows (before the fused kernel / two kernels / one, 2900 x 65 9.4 / 7.1 / 10.4, 3527 x 65 10.3 / 8.1 / 11.9, 4096 x 65 9.0 / 6.8 /
  // 12.4; even ones: 4096 x 16 8.0 / 6.2 / 6.8, 3527 x 300 12.3 / 9.5 / 8.9; 3000 x 2001 15.5 / - / 11.5).
  if (V == 8 && per % 2 != 0 && inner > 64 * V * 5 && per * batch < 512) return false;
  // A strip costs what it costs however short its rows (softmax, 2.4 to 4 ns), and the two kernels write no more for
  // short ones: rows of up to 16 elements only while the chip holds about all strips at once, of up to 31 while the
  // launches are most of the time.  bf16 softmax, two kernels / one, us: 40000 columns of 3 5.4 / 5.7 (eager calls 7.0 / 5.7), 65537 of 5
  // 6.5 / 7.2, 200000 of 3 8.1 / 19.0; batches 16 x 12 x 1500 7.1 / 6.9, 500 x 2 x 64 5.7 / 8.1, 4000 x 2 x 1500 104 / 515; 500 x
  // 24 x 300 14.3 / 14.2, 500 x 24 x 1500 31.8 / 54.9; 500 x 50 x 300 22.0 / 18.0.
  if (inner <= 16 && strips * batch > (batch > 1 ? 1250 + 25 * inner : 2100)) return false;
  if (inner < 32 && strips * batch > 6000) return false;
  LaunchRec& L = fp->launches[0];
  L.kid = K_ROW_XPOSE + (nv / 4 - 1) * 2 + (inner % V == 0 ? 1 : 0);
  L.block = (uint32_t)B;
  L.plan_kind = 1;
  L.rp.G = G;
  L.rp.log2G = ilog2_ceil(G);
  L.rp.nv = nv;
  L.rp.flags = ilog2_ceil(rpb / V);
  L.rp.rpb = rpb;
  fp->aux[0] = per;
  fp->aux[1] = strips;
  fp->aux[2] = strips * batch;
  fp->aux[3] = blocks / 8;
  L.grid[0] = (uint32_t)blocks;
  fp->pub.n_launches = 1;
  return true;
}

int resident_blocks(const disc_ctx* c, const Pattern& p, int kid, uint32_t block, uint32_t dyn_lds) {
  const int estimate = std::max(1, 16 / (int)((block + 63) / 64));
  if (c->device < 0 || kid < 0 || kid >= K_COUNT || !p.fn[kid]) return estimate;
  // the table is stepped in dynamic LDS: the question is asked for the upper end of the step
  const int bc = block <= 256 ? 0 : block <= 512 ? 1 : 2;
  const int step = (int)std::min<uint32_t>((dyn_lds + kLdsStep - 1) / kLdsStep, kLdsSteps - 1);
  int16_t& cell = p.resident[kid][bc][step];
  if (cell > 0) return cell;
  int nb = 0;
  if (hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(&nb, p.fn[kid], (int)block, (size_t)step * kLdsStep) != hipSuccess || nb < 1)
    nb = estimate;
  cell = (int16_t)nb;
  return nb;
}

void fill_args(const Pattern& p, const FullPlan& fp, const int64_t* dims, const void* const* in, void* const* outp,
               void* ws, unsigned char* buf) {
  const ShapeVals& sv = fp.sv;
  for (const auto& f : p.gen.args.fields) {
    unsigned char* dst = buf + f.offset;
    int64_t v = 0;
    switch (f.kind) {
      case ArgField::ROWS: v = sv.rows; memcpy(dst, &v, 8); break;
      case ArgField::INNER: v = sv.inner; memcpy(dst, &v, 8); break;
      case ArgField::NSLOTS: v = fp.nslots; memcpy(dst, &v, 8); break;
      case ArgField::SPR: v = fp.spr; memcpy(dst, &v, 8); break;
      case ArgField::MID: v = sv.mid; memcpy(dst, &v, 8); break;
      case ArgField::GROUP_SIZE: v = sv.group[f.index]; memcpy(dst, &v, 8); break;
      case ArgField::IN_PTR: memcpy(dst, &in[f.index], 8); break;
      case ArgField::OUT_PTR: memcpy(dst, &outp[f.index], 8); break;
      case ArgField::WS_PTR: { void* w = ws ? (char*)ws + fp.ws_off[f.index] : nullptr; memcpy(dst, &w, 8); break; }
      case ArgField::AUX: v = fp.aux[f.index]; memcpy(dst, &v, 8); break;
      case ArgField::STRIDE: v = sv.products[f.index]; memcpy(dst, &v, 8); break;
      case ArgField::DIMI: v = dims[p.an.dim_size_syms[f.index]]; memcpy(dst, &v, 8); break;
      case ArgField::SPR_DIV: { FastDivHost d = make_fastdiv((uint64_t)fp.spr); memcpy(dst, &d, 16); break; }
      case ArgField::GROUP_DIV: { FastDivHost d = make_fastdiv((uint64_t)sv.group[f.index]); memcpy(dst, &d, 16); break; }
      case ArgField::DIMF: { float x = (float)dims[p.an.dim_size_syms[f.index]]; memcpy(dst, &x, 4); break; }
    }
  }
}

const char* kUtilSource = R"SRC(
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ void copy_body(u32x4* __restrict__ dst, const u32x4* __restrict__ src, long long n) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + 3 * stride < n; i += 4 * stride) {
    u32x4 a, b, c, d;
    if constexpr (NT) {
      a = __builtin_nontemporal_load(src + i); b = __builtin_nontemporal_load(src + i + stride);
      c = __builtin_nontemporal_load(src + i + 2 * stride); d = __builtin_nontemporal_load(src + i + 3 * stride);
      __builtin_nontemporal_store(a, dst + i); __builtin_nontemporal_store(b, dst + i + stride);
      __builtin_nontemporal_store(c, dst + i + 2 * stride); __builtin_nontemporal_store(d, dst + i + 3 * stride);
    } else {
      a = src[i]; b = src[i + stride]; c = src[i + 2 * stride]; d = src[i + 3 * stride];
      dst[i] = a; dst[i + stride] = b; dst[i + 2 * stride] = c; dst[i + 3 * stride] = d;
    }
  }
  for (; i < n; i += stride) dst[i] = src[i];
}
extern "C" __global__ void __launch_bounds__(256) disc_util_copy_k(u32x4* __restrict__ dst, const u32x4* __restrict__ src, long long n) {
  copy_body<false>(dst, src, n);
}
extern "C" __global__ void __launch_bounds__(256) disc_util_copy_nt_k(u32x4* __restrict__ dst, const u32x4* __restrict__ src, long long n) {
  copy_body<true>(dst, src, n);
}
extern "C" __global__ void disc_util_empty_k() {}

// Streaming probes with the traffic mix of the row kernels and no arithmetic to speak of: per slot of
// eight 2-byte elements, KIND 0 reads 16 bytes + 8 bytes of a 1-byte stream and writes 16 bytes (3 bytes
// read : 2 written per element, the mix of the 12-op pattern), KIND 1 reads 16 + 16 bytes and writes 16
// (4 : 2, residual + LayerNorm).  NT = non-temporal accesses, U = slots in flight per lane.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <int KIND, bool NT, int U>
__device__ __forceinline__ void mix_body(u32x4* __restrict__ out, const u32x4* __restrict__ a, const u32x4* __restrict__ b,
                                         const u32x2* __restrict__ m, long long n) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x; i0 < n; i0 += stride * U) {
    u32x4 x[U], y[U];
    u32x2 k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long i = i0 + u * stride;
      if (i < n) {
        if constexpr (NT) x[u] = __builtin_nontemporal_load(a + i); else x[u] = a[i];
        if constexpr (KIND == 0) { if constexpr (NT) k[u] = __builtin_nontemporal_load(m + i); else k[u] = m[i]; }
        else { if constexpr (NT) y[u] = __builtin_nontemporal_load(b + i); else y[u] = b[i]; }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long i = i0 + u * stride;
      if (i < n) {
        u32x4 r = x[u];
        if constexpr (KIND == 0) { r.x ^= k[u].x; r.z ^= k[u].y; } else { r ^= y[u]; }
        if constexpr (NT) __builtin_nontemporal_store(r, out + i); else out[i] = r;
      }
    }
  }
}
#define DISC_MIX(KIND, NT, U)                                                                                        \
  extern "C" __global__ void __launch_bounds__(256) disc_util_mix_##KIND##_##NT##_##U(                               \
      u32x4* __restrict__ out, const u32x4* __restrict__ a, const u32x4* __restrict__ b, const u32x2* __restrict__ m, \
      long long n) {                                                                                                 \
    mix_body<KIND, NT != 0, U>(out, a, b, m, n);                                                                     \
  }
DISC_MIX(0, 0, 1) DISC_MIX(0, 0, 2) DISC_MIX(0, 0, 4) DISC_MIX(0, 0, 8)
DISC_MIX(0, 1, 1) DISC_MIX(0, 1, 2) DISC_MIX(0, 1, 4) DISC_MIX(0, 1, 8)
DISC_MIX(1, 0, 1) DISC_MIX(1, 0, 2) DISC_MIX(1, 0, 4) DISC_MIX(1, 0, 8)
DISC_MIX(1, 1, 1) DISC_MIX(1, 1, 2) DISC_MIX(1, 1, 4) DISC_MIX(1, 1, 8)
)SRC";

int ensure_util(disc_ctx* c) {
  if (c->util_module) return DISC_OK;
  if (c->device < 0) return set_err(c, DISC_ERR_INVALID_ARG, "host-only context");
  std::vector<char> code;
  double ms;
  int rc = compile_source(c, kUtilSource, &code, &ms);
  if (rc) return rc;
  hipError_t e = hipModuleLoadData(&c->util_module, code.data());
  if (e != hipSuccess) return hip_fail(c, e, "hipModuleLoadData");
  if ((e = hipModuleGetFunction(&c->util_copy, c->util_module, "disc_util_copy_k")) != hipSuccess) return hip_fail(c, e, "hipModuleGetFunction");
  if ((e = hipModuleGetFunction(&c->util_copy_nt, c->util_module, "disc_util_copy_nt_k")) != hipSuccess) return hip_fail(c, e, "hipModuleGetFunction");
  if ((e = hipModuleGetFunction(&c->util_empty, c->util_module, "disc_util_empty_k")) != hipSuccess) return hip_fail(c, e, "hipModuleGetFunction");
  for (int kind = 0; kind < 2; ++kind)
    for (int nt = 0; nt < 2; ++nt)
      for (int lu = 0; lu < 4; ++lu) {
        char name[48];
        snprintf(name, sizeof name, "disc_util_mix_%d_%d_%d", kind, nt, 1 << lu);
        if ((e = hipModuleGetFunction(&c->util_mix[kind][nt][lu], c->util_module, name)) != hipSuccess) return hip_fail(c, e, "hipModuleGetFunction");
      }
  return DISC_OK;
}

}  // namespace

// accessors for scratch.hip (the one source file compiled as HIP: it owns the static device array)
namespace disc {
int context_device(const disc_ctx* ctx) { return ctx ? ctx->device : -1; }
int context_fail(disc_ctx* ctx, int code, const char* msg) {
  try {
    return set_err(ctx, code, msg);
  } catch (...) {
    return code;
  }
}
}  // namespace disc
extern "C" int disc_static_scratch_init(disc_ctx* ctx);

// ============================================================================================
// C ABI
// ============================================================================================
// Nothing may leave an extern "C" function by exception: registration allocates (strings, vectors,
// maps), and an allocation failure there must come back as a status like everything else.
static int guard_fail(disc_ctx* c, const char* what) noexcept {
  if (c) {
    try {
      c->err = std::string("internal error: ") + what;
    } catch (...) {
    }
  }
  return DISC_ERR_INTERNAL;
}
#define DISC_TRY try {
#define DISC_CATCH(c)                                                          \
  }                                                                            \
  catch (const std::bad_alloc&) { return guard_fail(c, "out of host memory"); } \
  catch (const std::exception& e) { return guard_fail(c, e.what()); }          \
  catch (...) { return guard_fail(c, "unknown exception"); }

extern "C" {

int disc_create(disc_ctx** out, int hip_device) {
  DISC_TRY
  if (!out) return DISC_ERR_INVALID_ARG;
  *out = nullptr;
  std::unique_ptr<disc_ctx> c(new (std::nothrow) disc_ctx);
  if (!c) return DISC_ERR_INVALID_ARG;
  c->device = hip_device;
  if (hip_device >= 0) {
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || hip_device >= n) return DISC_ERR_HIP;
    if (hipSetDevice(hip_device) != hipSuccess) return DISC_ERR_HIP;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, hip_device) != hipSuccess) return DISC_ERR_HIP;
    c->n_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    // the device address of the static scratch array (disc_launch_static_scratch), once per device
    if (disc_static_scratch_init(c.get()) != DISC_OK) return DISC_ERR_HIP;
  }
  *out = c.release();
  return DISC_OK;
  DISC_CATCH(nullptr)
}

void disc_destroy(disc_ctx* ctx) {
  if (!ctx) return;
  if (ctx->device >= 0) {
    for (auto& p : ctx->patterns)
      if (p->module) (void)hipModuleUnload(p->module);
    for (auto& p : ctx->fused)
      if (p->module) (void)hipModuleUnload(p->module);
    if (ctx->util_module) (void)hipModuleUnload(ctx->util_module);
  }
  delete ctx;
}

const char* disc_last_error(const disc_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

// Text of the DISC_STATIC_ARGS / DISC_STATIC_PLAN macros for one shape: every non-pointer member
// of the argument block and of the launch-plan struct becomes an assignment of its constant.
static std::string static_macros(const Pattern& p, const FullPlan& fp, const int64_t* dims) {
  alignas(16) unsigned char buf[kArgBufBytes] = {0};
  std::vector<const void*> in(std::max(1, p.an.n_inputs), nullptr);
  std::vector<void*> outp(std::max(1, p.an.n_outputs), nullptr);
  fill_args(p, fp, dims, in.data(), outp.data(), nullptr, buf);
  std::ostringstream a;
  a << "#define DISC_STATIC_ARGS(A)";
  for (size_t i = 0; i < p.gen.args.fields.size(); ++i) {
    const ArgField& f = p.gen.args.fields[i];
    const std::string& n = p.gen.field_names[i];
    const unsigned char* src = buf + f.offset;
    switch (f.kind) {
      case ArgField::IN_PTR: case ArgField::OUT_PTR: case ArgField::WS_PTR: break;
      case ArgField::AUX:
        // the number of partial-sum rows follows the grid, which is chosen again at every launch
        // from the loaded kernel's residency: it stays a run-time argument
        if (p.gen.n_col_sums > 0 || p.gen.n_row_reds > 0) break;
        [[fallthrough]];
      default: {
        int64_t v;
        memcpy(&v, src, 8);
        a << " A." << n << " = " << v << "LL;";
        break;
      }
      case ArgField::SPR_DIV: case ArgField::GROUP_DIV: {
        uint32_t w[4];
        memcpy(w, src, 16);
        a << " A." << n << " = disc::FastDiv{" << w[0] << "u, " << w[1] << "u, " << w[2] << "u, 0u};";
        break;
      }
      case ArgField::DIMF: {
        uint32_t w;
        memcpy(&w, src, 4);
        a << " A." << n << " = __builtin_bit_cast(float, " << w << "u);";
        break;
      }
    }
  }
  a << "\n#define DISC_STATIC_PLAN(rp)";
  const LaunchRec& L = fp.launches[0];
  if (L.plan_kind == 1) {
    // Planned for aligned operands.  Whether a large launch of ragged rows has non-temporal accesses and slots on
    // whole lines, on 16-byte boundaries or unshifted follows its own operands (mixed chain 131072 x 2047, 2 bytes off:
    // 303 us with lines, 274 without; aligned 255 either way).  In a small one the shift alone stays a constant: as an
    // argument it costs every launch more (9000 x 1023 10.8 us / 11.0) than it gives the misaligned ones.
    const int low = L.rp.flags & 3, shifted = low | 4 | fp.pub.vec_width << 8;
    a << " rp.G = " << L.rp.G << "; rp.log2G = " << L.rp.log2G << "; rp.nv = " << L.rp.nv << "; rp.flags = ";
    if (L.rp.flags & 8) a << "rp.flags & 8 ? " << L.rp.flags << " : rp.flags & 4 ? " << shifted << " : " << low;
    else a << L.rp.flags;
    a << "; rp.rpb = " << L.rp.rpb << ";";
  } else if (L.plan_kind == 2)
    a << " rp.GC = " << L.cp.GC << "; rp.log2GC = " << L.cp.log2GC << "; rp.nchunk = " << L.cp.nchunk << "; rp.chunk_rows = "
      << L.cp.chunk_rows << "LL; rp.outer = " << L.cp.outer << "LL; rp.epi_rows = " << L.cp.epi_rows << "LL;";
  a << "\n";
  return a.str();
}

// compiles the pattern's generated source and looks its kernels up
static int load_module(disc_ctx* ctx, Pattern* p) {
  std::vector<char> code;
  const int rc = compile_source(ctx, p->gen.source, &code, &p->compile_ms);
  p->compile_events = 1;
  ctx->stats.compile_events++;
  if (rc) return rc;
  if (ctx->device >= 0) {
    hipError_t e = hipModuleLoadData(&p->module, code.data());
    if (e != hipSuccess) return hip_fail(ctx, e, "hipModuleLoadData");
    for (const auto& name : p->gen.kernels) {
      hipFunction_t f;
      e = hipModuleGetFunction(&f, p->module, (p->gen.prefix + name).c_str());
      if (e != hipSuccess) return hip_fail(ctx, e, ("hipModuleGetFunction " + name).c_str());
      const int kid = kernel_id(name);
      if (kid < 0) return set_err(ctx, DISC_ERR_COMPILE, "generated module holds an unnumbered kernel: " + name);
      p->fn[kid] = f;
    }
  }
  return DISC_OK;
}

static int register_impl(disc_ctx* ctx, const disc_op* ops, int n_ops, const disc_constraint* cs, int n_cs,
                         const int64_t* static_dims, int n_static_dims, int32_t* pattern_id_out) {
  if (!ctx) return DISC_ERR_INVALID_ARG;
  if (!pattern_id_out) return set_err(ctx, DISC_ERR_INVALID_ARG, "pattern_id_out is null");
  *pattern_id_out = -1;
  if (!ops || n_ops <= 0) return set_err(ctx, DISC_ERR_INVALID_ARG, "empty op list");
  if (n_cs < 0 || (n_cs > 0 && !cs)) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad constraint list");
  if (n_ops > DISC_MAX_OPS) return set_err(ctx, DISC_ERR_BAD_PATTERN, "too many ops");
  // pattern cache: the key is the op sequence and the constraints -- no sizes (Section 2)
  std::string key;
  for (int i = 0; i < n_ops; ++i) {
    disc_op o = ops[i];
    const int rank = std::max(0, std::min<int>(o.rank, DISC_MAX_RANK));
    for (int k = rank; k < DISC_MAX_RANK; ++k) o.dim[k] = 0;
    const bool uses_map = o.opcode == DISC_BROADCAST || o.opcode == DISC_DIM_SIZE ||
                          (o.opcode >= DISC_REDUCE_SUM && o.opcode <= DISC_REDUCE_ARGMAX);
    if (!uses_map) memset(o.axis_map, 0, sizeof o.axis_map);
    if (o.opcode != DISC_CONST) o.fconst = 0;
    key.append(reinterpret_cast<const char*>(&o.opcode), sizeof(int32_t) * 2);
    key.append(reinterpret_cast<const char*>(o.in), sizeof o.in);
    key.append(reinterpret_cast<const char*>(&o.rank), sizeof(int32_t));
    key.append(reinterpret_cast<const char*>(o.dim), sizeof o.dim);
    key.append(reinterpret_cast<const char*>(o.axis_map), sizeof o.axis_map);
    key.append(reinterpret_cast<const char*>(&o.fconst), sizeof o.fconst);
  }
  key.append("|");
  for (int i = 0; i < n_cs; ++i) key.append(reinterpret_cast<const char*>(&cs[i]), sizeof(disc_constraint));
  if (static_dims) {   // a single-shape module is a pattern of its own, one per shape
    key.append("|static");
    key.append(reinterpret_cast<const char*>(static_dims), sizeof(int64_t) * (size_t)n_static_dims);
  }
  auto hit = ctx->cache.find(key);
  if (hit != ctx->cache.end()) {
    *pattern_id_out = hit->second;
    ctx->stats.pattern_cache_hits++;
    return DISC_OK;
  }

  std::unique_ptr<Pattern> p(new Pattern);
  p->key = key;
  std::string err;
  int rc = analyze(ops, n_ops, cs, n_cs, &p->an, &err);
  if (rc) return set_err(ctx, rc, err);
  const std::string prefix = "disc_p" + std::to_string(ctx->patterns.size()) + "_";
  rc = generate(p->an, prefix, &p->gen, &err);
  if (rc) return set_err(ctx, rc, err);
  p->gen.source = std::string(kDeviceHeader) + "\n" + p->gen.source;
  // the launch path works in fixed-size buffers (nothing is allocated per launch)
  if (p->an.products.size() + p->an.offsets.size() + 2 * p->an.windows.size() > (size_t)kMaxShapeValues)
    return set_err(ctx, DISC_ERR_UNFUSIBLE, "too many strided, sliced or padded operands in one pattern");
  if (p->gen.args.size + 48 > kArgBufBytes) return set_err(ctx, DISC_ERR_UNFUSIBLE, "kernel-argument block too large");

  // launch-time constraint recipes
  DimClasses& dc = p->an.classes;
  p->class_of_dim.assign(p->an.n_sym, 0);
  {
    std::map<int, int> rep_to_class;
    std::map<int, int> first_member;
    for (int d = 0; d < p->an.n_sym; ++d) {
      int r = dc.find(d);
      if (!rep_to_class.count(r)) rep_to_class[r] = (int)rep_to_class.size();
      p->class_of_dim[d] = rep_to_class[r];
      if (first_member.count(r)) p->eq_checks.push_back({first_member[r], d});
      else first_member[r] = d;
      if (dc.static_val[r] >= 0 && first_member[r] == d) p->static_checks.push_back({d, dc.static_val[r]});
    }
    p->n_classes = (int)rep_to_class.size();
  }
  // algorithmic bytes: every operand and result once; an input that is only read through slices
  // counts with the elements its slices read
  std::vector<char> read_whole(p->an.ops.size(), 0);
  for (const auto& op : p->an.ops) {
    if (op.opcode == DISC_SLICE || op.opcode <= DISC_DIM_SIZE) continue;   // (a PAD reads its operand whole)
    for (int k = 0; k < 3; ++k)
      if (op.in[k] >= 0 && (k == 0 || op.opcode == DISC_SELECT || (op.opcode >= DISC_ADD && op.opcode <= DISC_NE)))
        read_whole[op.in[k]] = 1;
  }
  for (size_t i = 0; i < p->an.ops.size(); ++i) {
    const disc_op& op = p->an.ops[i];
    if (op.opcode == DISC_PARAM && !read_whole[i]) continue;
    if (op.opcode == DISC_SLICE && read_whole[op.in[0]]) continue;
    if (op.opcode != DISC_PARAM && op.opcode != DISC_OUTPUT && op.opcode != DISC_SLICE) continue;
    DimProduct prod;
    for (int k = 0; k < op.rank; ++k) {
      if (op.dim[k] >= 0) prod.sym.push_back(op.dim[k]); else prod.stat *= -(int64_t)op.dim[k];
    }
    p->io_numel.push_back({prod, dtype_bytes(op.dtype)});
  }

  if (static_dims) {
    // plan the one shape with the generic rules, then regenerate the module with only the kernel
    // versions that plan launches and with every extent and plan member as a constant
    FullPlan fp;
    rc = make_plan(ctx, *p, static_dims, n_static_dims, -1, nullptr, nullptr, &fp, least_limit(*p));
    if (rc) return rc;
    GenOptions opt;
    for (int l = 0; l < fp.pub.n_launches; ++l) {
      const std::string k = kernel_name(fp.launches[l].kid);
      opt.only_kernels.push_back(k);
      // planned without pointers, i.e. for aligned operands: keep the plain sibling of a
      // non-temporal version for launches whose operands turn out not to be 16-byte aligned
      // (for a row kernel that sibling is the version for rows of whole slots, _e)
      if (k == "k_col_epi2_vec_nts") opt.only_kernels.push_back("k_col_epi2_vec");
      if (k.size() > 3 && k.compare(k.size() - 3, 3, "_nt") == 0)
        opt.only_kernels.push_back(k.substr(0, k.size() - 3) + (k.compare(0, 9, "k_row_vec") == 0 ? "_e" : ""));
    }
    if (opt.only_kernels.empty()) return set_err(ctx, DISC_ERR_SHAPE, "a single-shape pattern needs a shape that launches something");
    const std::string macros = static_macros(*p, fp, static_dims);
    Generated g2;
    rc = generate(p->an, prefix, &g2, &err, &opt);
    if (rc) return set_err(ctx, rc, err);
    g2.source = macros + std::string(kDeviceHeader) + "\n" + g2.source;
    p->gen = g2;
    p->is_static = true;
    p->static_dims.assign(static_dims, static_dims + n_static_dims);
  }
  rc = load_module(ctx, p.get());
  if (rc) return rc;
  const int id = (int)ctx->patterns.size();
  ctx->cache[key] = id;
  ctx->patterns.push_back(std::move(p));
  ctx->stats.patterns_registered++;
  *pattern_id_out = id;
  return DISC_OK;
}

int disc_register_pattern(disc_ctx* ctx, const disc_op* ops, int n_ops, const disc_constraint* cs, int n_cs,
                          int32_t* pattern_id_out) {
  DISC_TRY
  return register_impl(ctx, ops, n_ops, cs, n_cs, nullptr, 0, pattern_id_out);
  DISC_CATCH(ctx)
}

int disc_register_pattern_static(disc_ctx* ctx, const disc_op* ops, int n_ops, const disc_constraint* cs, int n_cs,
                                 const int64_t* dims, int n_dims, int32_t* pattern_id_out) {
  DISC_TRY
  if (!ctx) return DISC_ERR_INVALID_ARG;
  if (!dims || n_dims <= 0) return set_err(ctx, DISC_ERR_INVALID_ARG, "a single-shape pattern needs its dims");
  return register_impl(ctx, ops, n_ops, cs, n_cs, dims, n_dims, pattern_id_out);
  DISC_CATCH(ctx)
}

int disc_pattern_info(disc_ctx* ctx, int32_t id, disc_pattern_info_t* out) {
  DISC_TRY
  Pattern* p = get_pattern(ctx, id);
  if (!p || !out) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad pattern id or null output");
  memset(out, 0, sizeof *out);
  out->template_kind = p->an.tmpl;
  out->n_dims = p->an.n_sym;
  out->n_inputs = p->an.n_inputs;
  out->n_outputs = p->an.n_outputs;
  out->compile_events = p->compile_events;
  out->n_variants = (int)p->gen.kernels.size();
  out->n_phases = p->an.n_phases;
  out->vec_width = p->an.vec_width;
  out->n_collapsed = (int)p->an.groups.size();
  out->n_dim_classes = p->n_classes;
  for (int d = 0; d < p->an.n_sym && d < DISC_MAX_DIMS; ++d) out->dim_class[d] = p->class_of_dim[d];
  out->compile_ms = p->compile_ms;
  return DISC_OK;
  DISC_CATCH(ctx)
}

const char* disc_pattern_source(disc_ctx* ctx, int32_t id) {
  Pattern* p = get_pattern(ctx, id);
  return p ? p->gen.source.c_str() : nullptr;
}

int disc_workspace_bytes(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, size_t* out) {
  DISC_TRY
  Pattern* p = get_pattern(ctx, id);
  if (!p || !out) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad pattern id or null output");
  FullPlan fp;
  int rc = make_plan(ctx, *p, dims, n_dims, ctx->force_variant, nullptr, nullptr, &fp);   // same selection disc_launch will make
  if (rc) return rc;
  *out = fp.pub.workspace_bytes;
  return DISC_OK;
  DISC_CATCH(ctx)
}

int disc_plan(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, const void* const* inputs,
              void* const* outputs, int force_variant, disc_plan_t* out) {
  DISC_TRY
  Pattern* p = get_pattern(ctx, id);
  if (!p || !out) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad pattern id or null output");
  FullPlan fp;
  int rc = make_plan(ctx, *p, dims, n_dims, force_variant, inputs, outputs, &fp);
  if (rc) return rc;
  *out = fp.pub;
  return DISC_OK;
  DISC_CATCH(ctx)
}

int disc_force_variant(disc_ctx* ctx, int variant) {
  DISC_TRY
  if (!ctx || variant < -1 || variant >= DISC_V_COUNT) return set_err(ctx, DISC_ERR_INVALID_ARG, "unknown version");
  ctx->force_variant = variant;
  return DISC_OK;
  DISC_CATCH(ctx)
}

int disc_test_option(disc_ctx* ctx, int option, int value) {
  DISC_TRY
  if (!ctx) return DISC_ERR_INVALID_ARG;
  switch (option) {
    case DISC_OPT_NON_TEMPORAL: ctx->row_nt = value < 0 ? -1 : value > 0 ? 1 : 0; return DISC_OK;
    case DISC_OPT_STAGE_ROW_VECTORS: ctx->row_stage = value != 0; return DISC_OK;
    case DISC_OPT_ROW_ROUNDS: ctx->row_rounds = std::max(0, value); return DISC_OK;
    case DISC_OPT_ALIGN_ROW_SLOTS: ctx->row_shift = value != 0; return DISC_OK;
    case DISC_OPT_COMPACT_LOOKS: ctx->compact_looks = std::max(-1, value); return DISC_OK;
    default: return set_err(ctx, DISC_ERR_INVALID_ARG, "unknown option");
  }
  DISC_CATCH(ctx)
}

// the planned launches of one call
static int submit(disc_ctx* ctx, const Pattern* p, const FullPlan& fp, const int64_t* dims, const void* const* inputs,
                  void* const* outputs, void* workspace, void* hip_stream) {
  alignas(16) unsigned char buf[kArgBufBytes];
  const int asz = p->gen.args.size;   // (fits: checked at registration)
  fill_args(*p, fp, dims, inputs, outputs, workspace, buf);
  for (int l = 0; l < fp.pub.n_launches; ++l) {
    const LaunchRec& L = fp.launches[l];
    const hipFunction_t fn = L.kid >= 0 && L.kid < K_COUNT ? p->fn[L.kid] : nullptr;
    if (!fn) return set_err(ctx, DISC_ERR_HIP, std::string("kernel version missing: ") + kernel_name(L.kid));
    size_t size = (size_t)asz;
    if (L.plan_kind == 1) {
      memcpy(buf + asz, &L.rp, sizeof L.rp);
      size += sizeof L.rp;
    } else if (L.plan_kind == 2) {
      memcpy(buf + asz, &L.cp, sizeof L.cp);
      size += sizeof L.cp;
    }
    void* extra[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, buf, HIP_LAUNCH_PARAM_BUFFER_SIZE, &size, HIP_LAUNCH_PARAM_END};
    hipError_t e = hipModuleLaunchKernel(fn, L.grid[0], L.grid[1], L.grid[2], L.block, 1, 1, L.dyn_lds,
                                         (hipStream_t)hip_stream, nullptr, extra);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipModuleLaunchKernel");
    ctx->stats.device_launches++;
  }
  return DISC_OK;
}

// own_need: the workspace has to hold what this launch uses (the static scratch array), not what
// disc_workspace_bytes gives for operands of any alignment (a caller's workspace).
static int launch_impl(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, const void* const* inputs, int n_in,
                       void* const* outputs, int n_out, void* workspace, size_t workspace_bytes, void* hip_stream, bool own_need) {
  const int64_t t0 = now_ns();
  Pattern* p = get_pattern(ctx, id);
  if (!p) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad pattern id");
  if (ctx->device < 0) return set_err(ctx, DISC_ERR_INVALID_ARG, "host-only context cannot launch");
  if (n_in != p->an.n_inputs || n_out != p->an.n_outputs) {
    char buf[96];
    snprintf(buf, sizeof buf, "pattern takes %d inputs and %d outputs, got %d and %d", p->an.n_inputs, p->an.n_outputs, n_in, n_out);
    return set_err(ctx, DISC_ERR_INVALID_ARG, buf);
  }
  if ((n_in > 0 && !inputs) || !outputs) return set_err(ctx, DISC_ERR_INVALID_ARG, "null pointer array");
  FullPlan fp;
  // (a column reduce that could do without a workspace does, if there is none; with the static array always, so
  // that a call that can do without the shared array leaves it alone)
  const bool without = least_limit(*p) == 0;
  const size_t limit = own_need ? (without ? 0 : workspace_bytes) : workspace && without ? workspace_bytes : least_limit(*p);
  int rc = make_plan(ctx, *p, dims, n_dims, ctx->force_variant, inputs, outputs, &fp, limit);
  const int64_t t1 = now_ns();
  ctx->stats.host_plan_ns += t1 - t0;
  if (rc) return rc;
  if (fp.pub.n_launches == 0) {
    ctx->stats.launch_calls++;
    ctx->stats.host_launch_ns += now_ns() - t0;
    return DISC_OK;
  }
  for (int i = 0; i < n_in; ++i)
    if (!inputs[i]) return set_err(ctx, DISC_ERR_INVALID_ARG, "null input pointer");
  for (int i = 0; i < n_out; ++i)
    if (!outputs[i]) return set_err(ctx, DISC_ERR_INVALID_ARG, "null output pointer");
  const size_t need = own_need && fp.ws_need > 0 ? fp.ws_need : fp.pub.workspace_bytes;
  if (need > 0 && (!workspace || workspace_bytes < need))
    return set_err(ctx, DISC_ERR_WORKSPACE, "workspace missing or too small");

  rc = submit(ctx, p, fp, dims, inputs, outputs, workspace, hip_stream);
  if (rc) return rc;
  ctx->stats.launch_calls++;
  if (fp.pub.variant >= 0 && fp.pub.variant < DISC_V_COUNT) ctx->stats.variant_count[fp.pub.variant]++;
  ctx->stats.host_launch_ns += now_ns() - t0;
  return DISC_OK;
}

int disc_launch(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, const void* const* inputs, int n_in,
                void* const* outputs, int n_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  DISC_TRY
  return launch_impl(ctx, id, dims, n_dims, inputs, n_in, outputs, n_out, workspace, workspace_bytes, hip_stream, false);
  DISC_CATCH(ctx)
}

}  // extern "C"
namespace disc {
// scratch.hip: what a launch with these operands uses, and the launch itself, with the static array
int launch_need(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, const void* const* inputs, int n_in,
                void* const* outputs, int n_out, size_t* need) {
  DISC_TRY
  Pattern* p = get_pattern(ctx, id);
  if (!p) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad pattern id or null output");
  // (the launch itself refuses operands that do not match the pattern)
  const bool match = n_in == p->an.n_inputs && n_out == p->an.n_outputs;
  FullPlan fp;
  int rc = make_plan(ctx, *p, dims, n_dims, ctx->force_variant, match ? inputs : nullptr, match ? outputs : nullptr, &fp,
                     std::min<size_t>(least_limit(*p), DISC_STATIC_SCRATCH_BYTES));
  if (rc) return rc;
  *need = fp.ws_need > 0 ? fp.ws_need : fp.pub.workspace_bytes;
  return DISC_OK;
  DISC_CATCH(ctx)
}
int launch_scratch(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, const void* const* inputs, int n_in,
                   void* const* outputs, int n_out, void* scratch, size_t bytes, void* hip_stream) {
  DISC_TRY
  return launch_impl(ctx, id, dims, n_dims, inputs, n_in, outputs, n_out, scratch, bytes, hip_stream, true);
  DISC_CATCH(ctx)
}
}  // namespace disc
extern "C" {

int disc_get_stats(disc_ctx* ctx, disc_stats_t* out) {
  DISC_TRY
  if (!ctx || !out) return DISC_ERR_INVALID_ARG;
  *out = ctx->stats;
  return DISC_OK;
  DISC_CATCH(ctx)
}

static int util_copy_impl(disc_ctx* ctx, void* dst, const void* src, size_t bytes, void* hip_stream, bool nt) {
  if (!ctx || !dst || !src || (bytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15))
    return set_err(ctx, DISC_ERR_INVALID_ARG, "copy needs 16-byte aligned pointers and size");
  int rc = ensure_util(ctx);
  if (rc) return rc;
  long long n = (long long)(bytes / 16);
  if (n == 0) return DISC_OK;
  void* args[] = {&dst, &src, &n};
  long long blocks = std::min<long long>((n + 1023) / 1024, (long long)ctx->n_cus * 2);
  hipError_t e = hipModuleLaunchKernel(nt ? ctx->util_copy_nt : ctx->util_copy, (uint32_t)blocks, 1, 1, 256, 1, 1, 0,
                                       (hipStream_t)hip_stream, args, nullptr);
  return e == hipSuccess ? DISC_OK : hip_fail(ctx, e, "hipModuleLaunchKernel");
}

int disc_util_copy(disc_ctx* ctx, void* dst, const void* src, size_t bytes, void* hip_stream) {
  DISC_TRY
  return util_copy_impl(ctx, dst, src, bytes, hip_stream, false);
  DISC_CATCH(ctx)
}

int disc_util_copy_nt(disc_ctx* ctx, void* dst, const void* src, size_t bytes, void* hip_stream) {
  DISC_TRY
  return util_copy_impl(ctx, dst, src, bytes, hip_stream, true);
  DISC_CATCH(ctx)
}

int disc_util_mix(disc_ctx* ctx, int kind, int non_temporal, int slots_in_flight, int blocks_per_cu, void* out, const void* a,
                  const void* b_or_mask, size_t n_elems, void* hip_stream) {
  DISC_TRY
  if (!ctx || !out || !a || !b_or_mask || (n_elems & 7) || kind < 0 || kind > 1 || blocks_per_cu < 1 || blocks_per_cu > 64 ||
      (((uintptr_t)out | (uintptr_t)a | (uintptr_t)b_or_mask) & 15))
    return set_err(ctx, DISC_ERR_INVALID_ARG, "mix probe: 16-byte aligned pointers, n_elems a multiple of 8, kind 0 or 1");
  int lu = 0;
  while (lu < 4 && (1 << lu) != slots_in_flight) ++lu;
  if (lu == 4) return set_err(ctx, DISC_ERR_INVALID_ARG, "mix probe: slots in flight must be 1, 2, 4 or 8");
  int rc = ensure_util(ctx);
  if (rc) return rc;
  long long n = (long long)(n_elems / 8);
  if (n == 0) return DISC_OK;
  const void* bp = kind == 1 ? b_or_mask : nullptr;
  const void* mp = kind == 0 ? b_or_mask : nullptr;
  void* args[] = {&out, &a, &bp, &mp, &n};
  const long long blocks = std::min<long long>((n + 255) / 256, (long long)ctx->n_cus * blocks_per_cu);
  hipError_t e = hipModuleLaunchKernel(ctx->util_mix[kind][non_temporal ? 1 : 0][lu], (uint32_t)blocks, 1, 1, 256, 1, 1, 0,
                                       (hipStream_t)hip_stream, args, nullptr);
  return e == hipSuccess ? DISC_OK : hip_fail(ctx, e, "hipModuleLaunchKernel");
  DISC_CATCH(ctx)
}

int disc_util_empty_launch(disc_ctx* ctx, void* hip_stream) {
  DISC_TRY
  if (!ctx) return DISC_ERR_INVALID_ARG;
  int rc = ensure_util(ctx);
  if (rc) return rc;
  hipError_t e = hipModuleLaunchKernel(ctx->util_empty, 1, 1, 1, 64, 1, 1, 0, (hipStream_t)hip_stream, nullptr, nullptr);
  return e == hipSuccess ? DISC_OK : hip_fail(ctx, e, "hipModuleLaunchKernel");
  DISC_CATCH(ctx)
}

}  // extern "C"

// =================================================================================================
// Op graphs (Section 4.3: fusion decision; Section 4.2.2: buffer management): a list of ops that
// need not be one fusible pattern is cut into consecutive fusion patterns with the SAME test the
// single-pattern path uses (the checker's shape propagation + constraints), and the values that
// cross pattern boundaries get buffers planned by lifetime, shared between values whose shapes
// are the same symbolic expression.
// =================================================================================================
namespace {

bool is_leaf(int opcode) { return opcode == DISC_PARAM || opcode == DISC_CONST || opcode == DISC_DIM_SIZE; }

int op_arity(const disc_op& o) { return operand_count(o.opcode); }

// The op list of the pattern that computes the graph ops `S` (ascending ids): operands produced
// outside S become PARAMs (scalar leaves are copied instead), values of S read outside S (by ops
// of other groups or by graph OUTPUTs) become OUTPUTs, constraints between values that both
// appear are carried over.
// `wanted` null (while the cut is still growing): every value read outside S counts as an output,
// also those that readers will recompute, so that a candidate always has an output.  For the
// patterns as registered, `wanted` marks the values other patterns really take in (their
// in_values, which includes what their recomputed cones read) and the graph outputs.
void build_sub_pattern(const Graph& g, const std::vector<int>& S, const std::vector<char>& in_S,
                       std::vector<disc_op>* sub, std::vector<disc_constraint>* sub_cs, std::vector<int>* in_values,
                       std::vector<int>* out_values, const std::vector<char>* wanted) {
  const bool final_cut = wanted != nullptr;
  std::map<int, int> id_of;   // graph value -> sub-pattern value
  sub->clear();
  sub_cs->clear();
  in_values->clear();
  out_values->clear();
  std::function<int(int)> operand = [&](int v) -> int {
    auto it = id_of.find(v);
    if (it != id_of.end()) return it->second;
    const disc_op& src = g.ops[v];
    disc_op o = src;
    if (src.opcode == DISC_CONST || src.opcode == DISC_DIM_SIZE) {
      for (int k = 0; k < 3; ++k) o.in[k] = -1;
    } else if (!is_leaf(src.opcode) && g.remat[v]) {
      // a cheap element-wise function of graph inputs computed by another pattern: computed again
      // here, from the inputs, instead of being written out and read back
      const int n = op_arity(src);
      for (int k = 0; k < n; ++k) o.in[k] = operand(src.in[k]);
    } else {               // a graph input or a value of another group: a PARAM of its type and shape
      o.opcode = DISC_PARAM;
      for (int k = 0; k < 3; ++k) o.in[k] = -1;
      for (int k = 0; k < DISC_MAX_RANK; ++k) o.axis_map[k] = 0;
      o.fconst = 0;
      in_values->push_back(v);
    }
    sub->push_back(o);
    id_of[v] = (int)sub->size() - 1;
    return id_of[v];
  };
  // consumers outside S
  std::vector<char> read_outside(g.ops.size(), 0);
  for (size_t i = 0; i < g.ops.size(); ++i) {
    if (in_S[i] || !g.needed[i]) continue;
    const disc_op& o = g.ops[i];
    if (is_leaf(o.opcode)) continue;
    const int n = op_arity(o);
    for (int k = 0; k < n; ++k)
      if (o.in[k] >= 0 && in_S[o.in[k]] && !final_cut) read_outside[o.in[k]] = 1;
  }
  if (final_cut)
    for (int v : S)
      if ((*wanted)[v]) read_outside[v] = 1;
  // ops of S that only fed readers which now recompute them are left out of the final pattern
  std::vector<char> live(g.ops.size(), final_cut ? 0 : 1);
  if (final_cut)
    for (size_t r = S.size(); r-- > 0;) {
      const int v = S[r];
      if (read_outside[v]) live[v] = 1;
      if (!live[v]) continue;
      const int n = op_arity(g.ops[v]);
      for (int k = 0; k < n; ++k)
        if (in_S[g.ops[v].in[k]]) live[g.ops[v].in[k]] = 1;
    }
  for (int v : S) {
    if (!live[v]) continue;
    disc_op o = g.ops[v];
    const int n = op_arity(o);
    for (int k = 0; k < n; ++k) o.in[k] = operand(g.ops[v].in[k]);
    sub->push_back(o);
    id_of[v] = (int)sub->size() - 1;
  }
  for (int v : S)
    if (read_outside[v]) {
      disc_op o = g.ops[v];
      o.opcode = DISC_OUTPUT;
      o.in[0] = id_of[v];
      o.in[1] = o.in[2] = -1;
      for (int k = 0; k < DISC_MAX_RANK; ++k) o.axis_map[k] = 0;
      o.fconst = 0;
      sub->push_back(o);
      out_values->push_back(v);
    }
  for (const auto& c : g.cs) {
    auto a = id_of.find(c.a_value), b = id_of.find(c.b_value);
    if (a == id_of.end() || b == id_of.end()) continue;
    disc_constraint t = c;
    t.a_value = a->second;
    t.b_value = b->second;
    sub_cs->push_back(t);
  }
}

// bytes of value v at these dims; false when the product does not fit 2^62
bool value_bytes(const Graph& g, int v, const int64_t* dims, int64_t* out) {
  const disc_op& o = g.ops[v];
  int64_t n = dtype_bytes(o.dtype);
  for (int k = 0; k < o.rank; ++k)
    if (mul_ovf(n, o.dim[k] >= 0 ? dims[o.dim[k]] : -(int64_t)o.dim[k], &n)) return false;
  *out = n;
  return n < (1ll << 62);
}

Graph* get_graph(disc_ctx* ctx, int32_t id) {
  if (!ctx || id < 0 || id >= (int)ctx->graphs.size()) return nullptr;
  return ctx->graphs[id].get();
}

// byte offset of every buffer and of the shared pattern-workspace region for one set of dims
// buf_off: room for one offset per buffer (at most DISC_MAX_OPS)
// least: what the patterns cannot do without, instead of what they ask for
int graph_layout(disc_ctx* ctx, const Graph& g, const int64_t* dims, int n_dims, bool least, size_t* buf_off,
                 size_t* pattern_ws_off, size_t* total) {
  if (!dims || n_dims != g.n_sym) return set_err(ctx, DISC_ERR_INVALID_ARG, "wrong number of dims for this graph");
  for (int i = 0; i < n_dims; ++i)
    if (dims[i] < 0) return set_err(ctx, DISC_ERR_SHAPE, "negative dim");
  size_t off = 0;
  for (size_t b = 0; b < g.buffer_value.size(); ++b) {
    buf_off[b] = off;
    int64_t bytes = 0;
    if (!value_bytes(g, g.buffer_value[b], dims, &bytes) || off + (size_t)bytes + 256 < off)
      return set_err(ctx, DISC_ERR_SHAPE, "buffer size overflows");
    off += ((size_t)bytes + 255) / 256 * 256;
  }
  *pattern_ws_off = off;
  size_t need = 0;
  for (const auto& gr : g.groups) {
    const Pattern& p = *ctx->patterns[gr.pattern_id];
    FullPlan fp;
    const int rc = make_plan(ctx, p, dims, p.an.n_sym, ctx->force_variant, nullptr, nullptr, &fp, least ? least_limit(p) : SIZE_MAX);
    if (rc) return rc;
    need = std::max(need, fp.pub.workspace_bytes);
  }
  *total = off + need;
  return DISC_OK;
}

}  // namespace

// The module of row reduce `base` with its input `access` transposed; null when it cannot be had.
static std::unique_ptr<Pattern> fused_module(disc_ctx* ctx, const Pattern& base, int access) {
  std::unique_ptr<Pattern> p(new Pattern);
  p->an = base.an;
  p->eq_checks = base.eq_checks;
  p->static_checks = base.static_checks;
  p->class_of_dim = base.class_of_dim;
  p->n_classes = base.n_classes;
  p->io_numel = base.io_numel;
  GenOptions opt;
  opt.xpose_access = access;
  std::string err;
  if (generate(p->an, "disc_x" + std::to_string(ctx->fused.size()) + "_", &p->gen, &err, &opt)) return nullptr;
  p->gen.source = std::string(kDeviceHeader) + "\n" + p->gen.source;
  const std::string before = ctx->err;
  if (load_module(ctx, p.get())) {
    ctx->err = before;
    if (p->module) (void)hipModuleUnload(p->module);
    return nullptr;
  }
  return p;
}

// Group gi is a transpose whose result only the row reduce behind it reads: a second module of that row
// reduce, whose kernels read the transpose's operand.  Which route a call takes is decided per shape; without
// the module every call takes both patterns.
static void register_fused(disc_ctx* ctx, Graph& g, size_t gi) {
  const GraphGroup& t = g.groups[gi];
  GraphGroup& r = g.groups[gi + 1];
  if (ctx->patterns[t.pattern_id]->an.tmpl != DISC_TEMPLATE_TRANSPOSE || t.in_place.size() != 1 || t.out_values.size() != 1) return;
  const int v = t.out_values[0];
  const auto inter = g.inter_of_value.find(v);
  if (inter == g.inter_of_value.end() || g.inter[inter->second].last != (int)gi + 1) return;
  int input = -1;
  for (size_t k = 0; k < r.in_values.size(); ++k)
    if (r.in_values[k] == v) input = (int)k;
  // (the operand is read while the results are written: it must not lie in a buffer that they reuse)
  if (t.in_place[0].first == 2)
    for (const auto& o : r.out_place)
      if (o == t.in_place[0]) return;
  const Pattern& base = *ctx->patterns[r.pattern_id];
  const int access = input < 0 ? -1 : xpose_access(base.an, input);
  if (access < 0) return;
  const std::pair<int, int> key{r.pattern_id, input};
  auto known = ctx->fused_of.find(key);
  if (known == ctx->fused_of.end()) {
    std::unique_ptr<Pattern> p = fused_module(ctx, base, access);
    known = ctx->fused_of.emplace(key, p ? (int)ctx->fused.size() : -1).first;
    if (p) ctx->fused.push_back(std::move(p));
  }
  r.fused = known->second;
  r.fused_input = input;
}

// The plan of group r with the transpose in front of it (group t) in the same kernel.  `taken`: false when such a
// call goes through both patterns.
static int plan_fused(disc_ctx* ctx, const GraphGroup& t, const GraphGroup& r, const int64_t* dims, FullPlan* fp, bool* taken) {
  *taken = false;
  if (ctx->force_variant >= 0) return DISC_OK;
  const Pattern& tp = *ctx->patterns[t.pattern_id];
  const Pattern& p = *ctx->fused[r.fused];
  ShapeVals tv;
  int rc = shape_calc(ctx, tp, dims, tp.an.n_sym, &tv);
  if (rc) return rc;
  rc = shape_calc(ctx, p, dims, p.an.n_sym, &fp->sv);
  if (rc) return rc;
  const int ng = (int)tp.an.groups.size();
  const int64_t per = tv.group[ng - 2], batch = ng == 3 ? tv.group[0] : 1;
  if (fp->sv.rows == 0 || fp->sv.inner == 0 || fp->sv.rows != batch * per || fp->sv.inner != tv.group[ng - 1]) return DISC_OK;
  *taken = plan_xpose(ctx, per, batch, fp->sv.inner, p.an.vec_width, fp);
  return DISC_OK;
}

// Its launch, unless the results lie over the operand.
static int launch_fused(disc_ctx* ctx, const GraphGroup& t, const GraphGroup& r, const int64_t* dims, const void* const* in,
                        void* const* outp, void* hip_stream, bool* taken) {
  *taken = false;
  const int64_t t0 = now_ns();
  if (ctx->device < 0) return DISC_OK;
  const Pattern& p = *ctx->fused[r.fused];
  FullPlan fp;
  bool one = false;
  int rc = plan_fused(ctx, t, r, dims, &fp, &one);
  if (rc || !one) return rc;
  const char* lo = static_cast<const char*>(in[r.fused_input]);
  const char* hi = lo + fp.sv.rows * fp.sv.inner * dtype_bytes(ctx->patterns[t.pattern_id]->an.accesses[0].dtype);
  for (const Access& a : p.an.accesses) {      // (through both patterns the operand was read before anything was written)
    if (!a.is_output) continue;
    const char* o = static_cast<const char*>(outp[a.slot]);
    if (o < hi && lo < o + fp.sv.rows * (a.has_inner ? fp.sv.inner : 1) * dtype_bytes(a.dtype)) return DISC_OK;
  }
  ctx->stats.host_plan_ns += now_ns() - t0;
  rc = submit(ctx, &p, fp, dims, in, outp, nullptr, hip_stream);
  if (rc) return rc;
  *taken = true;
  ctx->stats.launch_calls++;
  ctx->stats.host_launch_ns += now_ns() - t0;
  return DISC_OK;
}

int disc_register_graph(disc_ctx* ctx, const disc_op* ops, int n_ops, const disc_constraint* cs, int n_cs,
                        int32_t* graph_id_out) {
  DISC_TRY
  if (!ctx) return DISC_ERR_INVALID_ARG;
  if (!graph_id_out) return set_err(ctx, DISC_ERR_INVALID_ARG, "graph_id_out is null");
  *graph_id_out = -1;
  if (!ops || n_ops <= 0) return set_err(ctx, DISC_ERR_INVALID_ARG, "empty op list");
  if (n_cs < 0 || (n_cs > 0 && !cs)) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad constraint list");
  if (n_ops > DISC_MAX_OPS) return set_err(ctx, DISC_ERR_BAD_PATTERN, "too many ops");
  std::unique_ptr<Graph> g(new Graph);
  g->ops.assign(ops, ops + n_ops);
  if (n_cs) g->cs.assign(cs, cs + n_cs);
  g->group_of_op.assign(n_ops, -1);
  // structure checks the per-pattern checker cannot make on a cut-up list
  std::vector<int> compute;
  for (int i = 0; i < n_ops; ++i) {
    const disc_op& o = g->ops[i];
    if (o.opcode < 0 || o.opcode >= DISC_OPCODE_COUNT) return set_err(ctx, DISC_ERR_BAD_PATTERN, "unknown opcode");
    if (o.rank < 0 || o.rank > DISC_MAX_RANK) return set_err(ctx, DISC_ERR_BAD_PATTERN, "rank out of range");
    const int n = op_arity(o);
    for (int k = 0; k < n; ++k)
      if (o.in[k] < 0 || o.in[k] >= i || g->ops[o.in[k]].opcode == DISC_OUTPUT)
        return set_err(ctx, DISC_ERR_BAD_PATTERN, "operand does not name an earlier value");
    for (int k = 0; k < o.rank; ++k)
      if (o.dim[k] >= 0) g->n_sym = std::max(g->n_sym, o.dim[k] + 1);
    if (o.opcode == DISC_DIM_SIZE) g->n_sym = std::max(g->n_sym, o.axis_map[0] + 1);
    if (o.opcode == DISC_SLICE || o.opcode == DISC_PAD)       // starts / low paddings that are runtime values
      for (int k = 0; k < o.rank; ++k) g->n_sym = std::max(g->n_sym, o.axis_map[k] + 1);
    if (o.opcode == DISC_PARAM) g->param_index[i] = g->n_inputs++;
    else if (o.opcode == DISC_OUTPUT) {
      if (n < 1 || is_leaf(g->ops[o.in[0]].opcode))
        return set_err(ctx, DISC_ERR_BAD_PATTERN, "a graph output must be a computed value");
      if (g->output_index.count(o.in[0])) return set_err(ctx, DISC_ERR_BAD_PATTERN, "a value is output twice");
      g->output_index[o.in[0]] = g->n_outputs++;
    } else if (!is_leaf(o.opcode)) compute.push_back(i);
  }
  if (g->n_sym > DISC_MAX_DIMS) return set_err(ctx, DISC_ERR_BAD_PATTERN, "too many symbolic dims");
  // dead code: ops that no graph output depends on belong to no pattern
  {
    std::vector<char>& needed = g->needed;
    needed.assign(n_ops, 0);
    for (int i = n_ops - 1; i >= 0; --i) {
      const disc_op& o = g->ops[i];
      if (o.opcode == DISC_OUTPUT) needed[i] = 1;
      if (!needed[i]) continue;
      const int n = op_arity(o);
      for (int k = 0; k < n; ++k) needed[o.in[k]] = 1;
    }
    std::vector<int> kept;
    for (int v : compute)
      if (needed[v]) kept.push_back(v);
    compute.swap(kept);
  }
  if (compute.empty() || g->n_outputs == 0) return set_err(ctx, DISC_ERR_BAD_PATTERN, "nothing to compute");

  // Recomputing instead of buffering.  A value that is a cheap element-wise function of at most
  // two graph inputs (a cast of an input, an input plus a broadcast bias, ...) does not cross
  // cuts: a pattern that reads it computes it again from the inputs, which costs no more traffic
  // than reading the stored result and saves writing it.  At level 2 the function may also use
  // reduction results (per-row or per-column values: small), so that e.g. normalised activations
  // are recomputed from the input and the row statistics instead of being stored in full; the
  // reduction results themselves then cross the cut as small buffers.  Level 1: inputs only.
  // Level 0: nothing is recomputed.  The highest level whose cut passes the checker is taken.
  auto compute_remat = [&](int level) {
    g->remat.assign(n_ops, 0);
    if (level == 0) return;
    std::vector<std::set<int>> cone_params(n_ops), cone_anchors(n_ops);
    std::vector<int> cone_ops(n_ops, 0);
    const size_t max_ops = level == 2 ? 16 : 8;
    for (int i = 0; i < n_ops; ++i) {
      const disc_op& o = g->ops[i];
      if (o.opcode == DISC_PARAM) { cone_params[i].insert(i); continue; }
      if (is_leaf(o.opcode) || o.opcode == DISC_OUTPUT) continue;
      if (o.opcode >= DISC_REDUCE_SUM && o.opcode <= DISC_REDUCE_ARGMAX) {
        if (level == 2) cone_anchors[i].insert(i);
        continue;
      }
      // a transpose that moves the innermost axis fuses with nothing: it stays a kernel of its own
      if (o.opcode == DISC_TRANSPOSE && o.rank > 0 && o.axis_map[o.rank - 1] != o.rank - 1) continue;
      bool ok = true;
      int nops = 1;
      const int n = op_arity(o);
      for (int k = 0; k < n && ok; ++k) {
        const int a = o.in[k];
        const bool anchor = level == 2 && g->ops[a].opcode >= DISC_REDUCE_SUM && g->ops[a].opcode <= DISC_REDUCE_ARGMAX;
        if (!is_leaf(g->ops[a].opcode) && !g->remat[a] && !anchor) ok = false;
        cone_params[i].insert(cone_params[a].begin(), cone_params[a].end());
        cone_anchors[i].insert(cone_anchors[a].begin(), cone_anchors[a].end());
        nops += cone_ops[a];
      }
      cone_ops[i] = nops;
      if (ok && cone_params[i].size() <= 2 && cone_anchors[i].size() <= 4 && (size_t)nops <= max_ops) g->remat[i] = 1;
    }
  };

  // greedy cut in list order: an op joins the current pattern when the checker still accepts the
  // pattern with it (one provable iteration space, one template); otherwise it opens the next one
  std::vector<disc_op> sub;
  std::vector<disc_constraint> sub_cs;
  std::vector<int> ins, outs;
  auto fusible = [&](const std::vector<int>& S, std::string* why) {
    std::vector<char> in_S(n_ops, 0);
    for (int v : S) in_S[v] = 1;
    build_sub_pattern(*g, S, in_S, &sub, &sub_cs, &ins, &outs, nullptr);
    Analysis an;
    return analyze(sub.data(), (int)sub.size(), sub_cs.empty() ? nullptr : sub_cs.data(), (int)sub_cs.size(), &an, why);
  };
  // The patterns as they will be registered, last to first: a pattern's outputs are the graph
  // outputs it computes and what later patterns take in -- directly or through the cones they
  // recompute.  `each` gets every pattern that has an output; returns the first failure.
  struct FinalPattern {
    std::vector<disc_op> ops;
    std::vector<disc_constraint> cs;
    std::vector<int> in_values, out_values;
  };
  auto finalize = [&](const std::vector<std::vector<int>>& cs_, std::vector<FinalPattern>* each, std::string* why) {
    std::vector<char> wanted(n_ops, 0);
    for (const auto& kv : g->output_index) wanted[kv.first] = 1;
    each->assign(cs_.size(), FinalPattern());
    for (size_t gi = cs_.size(); gi-- > 0;) {
      std::vector<char> in_S(n_ops, 0);
      for (int v : cs_[gi]) in_S[v] = 1;
      FinalPattern& fp = (*each)[gi];
      build_sub_pattern(*g, cs_[gi], in_S, &fp.ops, &fp.cs, &fp.in_values, &fp.out_values, &wanted);
      if (fp.out_values.empty()) { fp.in_values.clear(); continue; }      // nothing reads it: dropped
      for (int v : fp.in_values) wanted[v] = 1;
      Analysis an;
      const int rc = analyze(fp.ops.data(), (int)fp.ops.size(), fp.cs.empty() ? nullptr : fp.cs.data(), (int)fp.cs.size(), &an, why);
      if (rc) return rc;
    }
    return (int)DISC_OK;
  };
  std::vector<std::vector<int>> cuts;
  std::string why;
  int cut_rc = DISC_OK;
  for (int level = 2; level >= 0; --level) {
    compute_remat(level);
    cuts.clear();
    cut_rc = DISC_OK;
    std::vector<int> cur;
    for (int v : compute) {
      cur.push_back(v);
      if (fusible(cur, &why) == DISC_OK) continue;
      cur.pop_back();
      if (cur.empty()) {
        cut_rc = set_err(ctx, DISC_ERR_UNFUSIBLE, "op " + std::to_string(v) + " is not a pattern on its own: " + why);
        break;
      }
      cuts.push_back(cur);
      cur.assign(1, v);
      const int rc = fusible(cur, &why);
      if (rc) {
        cut_rc = set_err(ctx, rc, "op " + std::to_string(v) + " is not a pattern on its own: " + why);
        break;
      }
    }
    if (cut_rc == DISC_OK) {
      cuts.push_back(cur);
      std::vector<FinalPattern> probe;
      const int rc = finalize(cuts, &probe, &why);
      if (rc) cut_rc = set_err(ctx, rc, "a cut of the graph is not a pattern: " + why);
    }
    if (cut_rc == DISC_OK) break;
  }
  if (cut_rc != DISC_OK) return cut_rc;

  // Sinking: the greedy cut also pulls in ops that only feed the NEXT pattern (say the |x| ahead of
  // a reduction the current pattern cannot hold), which turns their result into one more buffer.
  // Such an op moves to the pattern of its users when nothing of its own pattern and no graph
  // output reads it, all its users sit in one later pattern, that pattern still passes the checker
  // with it, and each of its computed operands crosses a pattern boundary anyway -- then the move
  // saves one write and one read of the op's result and adds at most one read of an operand.
  {
    std::vector<int> grp(n_ops, -1);
    for (size_t gi = 0; gi < cuts.size(); ++gi)
      for (int v : cuts[gi]) grp[v] = (int)gi;
    std::vector<std::vector<int>> users(n_ops);
    for (int i = 0; i < n_ops; ++i) {
      if (is_leaf(g->ops[i].opcode) || !g->needed[i]) continue;
      const int n = op_arity(g->ops[i]);
      for (int k = 0; k < n; ++k) users[g->ops[i].in[k]].push_back(i);
    }
    auto read_elsewhere = [&](int v, int except) {       // graph output, or read outside its pattern by another op
      for (int u : users[v]) {
        if (u == except) continue;
        if (g->ops[u].opcode == DISC_OUTPUT || grp[u] != grp[v]) return true;
      }
      return false;
    };
    bool moved = true;
    while (moved) {
      moved = false;
      for (size_t gi = 0; gi + 1 < cuts.size(); ++gi) {
        for (size_t pos = cuts[gi].size(); pos-- > 0;) {
          const int x = cuts[gi][pos];
          if (users[x].empty()) continue;
          // a reduction stays where its operand is computed: moved, it would read the operand again
          if (g->ops[x].opcode >= DISC_REDUCE_SUM && g->ops[x].opcode <= DISC_REDUCE_ARGMAX) continue;
          int to = -1;
          bool ok = true;
          for (int u : users[x]) {
            if (g->ops[u].opcode == DISC_OUTPUT || grp[u] <= (int)gi) { ok = false; break; }
            if (to >= 0 && grp[u] != to) { ok = false; break; }
            to = grp[u];
          }
          if (!ok || to < 0) continue;
          const int n = op_arity(g->ops[x]);
          for (int k = 0; k < n && ok; ++k) {
            const int a = g->ops[x].in[k];
            if (!is_leaf(g->ops[a].opcode) && grp[a] == (int)gi && !read_elsewhere(a, x)) ok = false;
          }
          if (!ok) continue;
          std::vector<int> bigger = cuts[to];
          bigger.insert(std::lower_bound(bigger.begin(), bigger.end(), x), x);
          if (fusible(bigger, &why) != DISC_OK) continue;
          std::vector<int> smaller = cuts[gi];
          smaller.erase(smaller.begin() + (long)pos);
          if (!smaller.empty() && fusible(smaller, &why) != DISC_OK) continue;
          cuts[to].swap(bigger);
          cuts[gi].swap(smaller);
          grp[x] = to;
          moved = true;
        }
      }
    }
    std::vector<std::vector<int>> kept;
    for (auto& c : cuts)
      if (!c.empty()) kept.push_back(c);
    cuts.swap(kept);
  }
  if (cuts.size() > (size_t)DISC_MAX_GRAPH_PATTERNS) return set_err(ctx, DISC_ERR_BAD_PATTERN, "the graph needs too many patterns");

  std::vector<FinalPattern> finals;
  {
    const int rc = finalize(cuts, &finals, &why);
    if (rc) return set_err(ctx, rc, "a cut of the graph is not a pattern: " + why);
  }
  for (size_t gi = 0; gi < cuts.size(); ++gi) {
    GraphGroup gr;
    gr.ops = cuts[gi];
    for (int v : gr.ops) g->group_of_op[v] = (int)gi;
    gr.in_values = finals[gi].in_values;
    gr.out_values = finals[gi].out_values;
    if (gr.out_values.empty()) { gr.pattern_id = -1; g->groups.push_back(gr); continue; }   // dead code: nothing reads it
    int32_t pid = -1;
    int rc = disc_register_pattern(ctx, finals[gi].ops.data(), (int)finals[gi].ops.size(),
                                   finals[gi].cs.empty() ? nullptr : finals[gi].cs.data(), (int)finals[gi].cs.size(), &pid);
    if (rc) return rc;
    gr.pattern_id = pid;
    g->groups.push_back(gr);
  }
  // drop groups nothing reads
  {
    std::vector<GraphGroup> kept;
    std::vector<int> renum(g->groups.size(), -1);
    for (size_t gi = 0; gi < g->groups.size(); ++gi)
      if (g->groups[gi].pattern_id >= 0) { renum[gi] = (int)kept.size(); kept.push_back(g->groups[gi]); }
    for (int& x : g->group_of_op)
      if (x >= 0) x = renum[x];
    g->groups.swap(kept);
  }
  if (g->groups.empty()) return set_err(ctx, DISC_ERR_BAD_PATTERN, "no output depends on a computed value");

  // values that cross pattern boundaries and are not graph outputs live in planned buffers
  for (size_t gi = 0; gi < g->groups.size(); ++gi)
    for (int v : g->groups[gi].out_values) {
      if (g->output_index.count(v)) continue;
      GraphIntermediate it;
      it.value = v;
      it.first = it.last = (int)gi;
      g->inter_of_value[v] = (int)g->inter.size();
      g->inter.push_back(it);
    }
  for (size_t gi = 0; gi < g->groups.size(); ++gi)
    for (int v : g->groups[gi].in_values) {
      auto it = g->inter_of_value.find(v);
      if (it != g->inter_of_value.end()) g->inter[it->second].last = std::max(g->inter[it->second].last, (int)gi);
    }
  // a buffer is reused by a later value of the same dtype size and the same symbolic shape once
  // its previous tenant has been read for the last time (Section 4.2.2: reuse by shape compatibility)
  {
    std::vector<int> free_after;          // per buffer: last group that reads its tenant
    std::vector<std::string> key_of;      // per buffer
    for (auto& it : g->inter) {
      const disc_op& o = g->ops[it.value];
      std::string key(1, (char)dtype_bytes(o.dtype));
      key.append(reinterpret_cast<const char*>(o.dim), sizeof(int32_t) * (size_t)o.rank);
      int pick = -1;
      for (size_t b = 0; b < key_of.size() && pick < 0; ++b)
        if (key_of[b] == key && free_after[b] < it.first) pick = (int)b;
      if (pick < 0) {
        pick = (int)key_of.size();
        key_of.push_back(key);
        free_after.push_back(it.last);
        g->buffer_value.push_back(it.value);
      } else {
        free_after[pick] = it.last;
      }
      it.buffer = pick;
    }
  }
  // the launch path looks nothing up: every operand of every pattern gets its place now
  for (auto& gr : g->groups) {
    auto place_of = [&](int v) -> std::pair<int, int> {
      auto pi = g->param_index.find(v);
      if (pi != g->param_index.end()) return {0, pi->second};
      auto oi = g->output_index.find(v);
      if (oi != g->output_index.end()) return {1, oi->second};
      auto it = g->inter_of_value.find(v);
      if (it != g->inter_of_value.end()) return {2, g->inter[it->second].buffer};
      return {-1, 0};
    };
    for (int v : gr.in_values) gr.in_place.push_back(place_of(v));
    for (int v : gr.out_values) gr.out_place.push_back(place_of(v));
    for (const auto& pl : gr.in_place)
      if (pl.first < 0) return set_err(ctx, DISC_ERR_INTERNAL, "a value of the graph has no place");
    for (const auto& pl : gr.out_place)
      if (pl.first < 0) return set_err(ctx, DISC_ERR_INTERNAL, "a value of the graph has no place");
    if (gr.in_place.size() > (size_t)DISC_MAX_OPS || gr.out_place.size() > (size_t)DISC_MAX_OPS)
      return set_err(ctx, DISC_ERR_BAD_PATTERN, "too many operands in one pattern of the graph");
  }
  if (g->buffer_value.size() > (size_t)DISC_MAX_OPS) return set_err(ctx, DISC_ERR_BAD_PATTERN, "too many buffers");
  for (size_t gi = 0; gi + 1 < g->groups.size(); ++gi) register_fused(ctx, *g, gi);
  const int id = (int)ctx->graphs.size();
  ctx->graphs.push_back(std::move(g));
  *graph_id_out = id;
  return DISC_OK;
  DISC_CATCH(ctx)
}

int disc_graph_info(disc_ctx* ctx, int32_t id, disc_graph_info_t* out) {
  DISC_TRY
  Graph* g = get_graph(ctx, id);
  if (!g || !out) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad graph id or null output");
  memset(out, 0, sizeof *out);
  out->n_dims = g->n_sym;
  out->n_inputs = g->n_inputs;
  out->n_outputs = g->n_outputs;
  out->n_patterns = (int)g->groups.size();
  out->n_intermediates = (int)g->inter.size();
  out->n_buffers = (int)g->buffer_value.size();
  for (size_t i = 0; i < g->groups.size() && i < DISC_MAX_GRAPH_PATTERNS; ++i) {
    out->pattern_id[i] = g->groups[i].pattern_id;
    out->pattern_ops[i] = (int)g->groups[i].ops.size();
  }
  for (size_t i = 0; i < g->group_of_op.size() && i < DISC_MAX_OPS; ++i) out->group_of_op[i] = g->group_of_op[i];
  return DISC_OK;
  DISC_CATCH(ctx)
}

int disc_graph_workspace_bytes(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, size_t* out) {
  DISC_TRY
  Graph* g = get_graph(ctx, id);
  if (!g || !out) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad graph id or null output");
  size_t off[DISC_MAX_OPS];
  size_t pws = 0;
  return graph_layout(ctx, *g, dims, n_dims, false, off, &pws, out);
  DISC_CATCH(ctx)
}

int disc_graph_plan(disc_ctx* ctx, int32_t id, int pattern, const int64_t* dims, int n_dims, disc_plan_t* out) {
  DISC_TRY
  Graph* g = get_graph(ctx, id);
  if (!g || !out || pattern < 0 || pattern >= (int)g->groups.size())
    return set_err(ctx, DISC_ERR_INVALID_ARG, "bad graph id, pattern index or null output");
  if (!dims || n_dims != g->n_sym) return set_err(ctx, DISC_ERR_INVALID_ARG, "wrong number of dims for this graph");
  const size_t gi = (size_t)pattern;
  FullPlan fp;
  for (const bool second : {true, false}) {     // the row reduce of a fused pair, the transpose of one
    if (second ? gi == 0 : gi + 1 >= g->groups.size()) continue;
    const GraphGroup &t = g->groups[second ? gi - 1 : gi], &r = g->groups[second ? gi : gi + 1];
    if (r.fused < 0) continue;
    bool taken = false;
    const int rc = plan_fused(ctx, t, r, dims, &fp, &taken);
    if (rc) return rc;
    if (!taken) continue;
    memset(out, 0, sizeof *out);
    out->variant = -1;
    if (!second) return DISC_OK;
    const LaunchRec& L = fp.launches[0];
    out->rows = fp.sv.rows;
    out->inner = fp.sv.inner;
    out->algorithmic_bytes = fp.sv.alg_bytes;
    out->n_launches = 1;
    out->vec_width = ctx->fused[r.fused]->an.vec_width;
    out->index_bits = 64;
    out->lanes_per_row = L.rp.G;
    out->slots_per_lane = out->reg_slots = L.rp.nv;
    for (int k = 0; k < 3; ++k) out->grid[0][k] = L.grid[k];
    out->block[0][0] = L.block;
    out->block[0][1] = out->block[0][2] = 1;
    snprintf(out->kernel[0], sizeof out->kernel[0], "%s%s", ctx->fused[r.fused]->gen.prefix.c_str(), kernel_name(L.kid));
    return DISC_OK;
  }
  const Pattern& p = *ctx->patterns[g->groups[gi].pattern_id];
  return disc_plan(ctx, g->groups[gi].pattern_id, dims, p.an.n_sym, nullptr, nullptr, ctx->force_variant, out);
  DISC_CATCH(ctx)
}

int disc_graph_launch(disc_ctx* ctx, int32_t id, const int64_t* dims, int n_dims, const void* const* inputs, int n_in,
                      void* const* outputs, int n_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  DISC_TRY
  Graph* g = get_graph(ctx, id);
  if (!g) return set_err(ctx, DISC_ERR_INVALID_ARG, "bad graph id");
  if (n_in != g->n_inputs || n_out != g->n_outputs) return set_err(ctx, DISC_ERR_INVALID_ARG, "wrong number of inputs or outputs");
  if ((n_in > 0 && !inputs) || !outputs) return set_err(ctx, DISC_ERR_INVALID_ARG, "null pointer array");
  // nothing is allocated and nothing looked up here: offsets and pointer arrays live on the stack,
  // the place of every operand was resolved at registration
  size_t off[DISC_MAX_OPS];
  size_t pws = 0, total = 0;
  int rc = graph_layout(ctx, *g, dims, n_dims, false, off, &pws, &total);
  if (rc) return rc;
  if (!workspace) workspace_bytes = 0;
  if (workspace_bytes < total) {
    size_t least = 0;
    rc = graph_layout(ctx, *g, dims, n_dims, true, off, &pws, &least);
    if (rc) return rc;
    if (workspace_bytes < least) return set_err(ctx, DISC_ERR_WORKSPACE, "workspace missing or too small");
    total = std::max(pws, workspace_bytes);      // (the patterns get what is left behind the buffers)
  }
  char* ws = static_cast<char*>(workspace);
  const void* in[DISC_MAX_OPS];
  void* outp[DISC_MAX_OPS];
  auto where = [&](const std::pair<int, int>& pl) -> void* {
    return pl.first == 0 ? const_cast<void*>(inputs[pl.second]) : pl.first == 1 ? outputs[pl.second] : ws + off[pl.second];
  };
  for (size_t gi = 0; gi < g->groups.size(); ++gi) {
    const GraphGroup& gr = g->groups[gi];
    const GraphGroup* next = gi + 1 < g->groups.size() ? &g->groups[gi + 1] : nullptr;
    if (next && next->fused >= 0) {
      bool taken = true;
      for (size_t k = 0; k < next->in_place.size(); ++k) {
        in[k] = where(k == (size_t)next->fused_input ? gr.in_place[0] : next->in_place[k]);
        taken = taken && in[k];
      }
      for (size_t k = 0; k < next->out_place.size(); ++k) {
        outp[k] = where(next->out_place[k]);
        taken = taken && outp[k];
      }
      if (taken) {
        rc = launch_fused(ctx, gr, *next, dims, in, outp, hip_stream, &taken);
        if (rc) return rc;
        if (taken) {
          ++gi;
          continue;
        }
      }
    }
    const int ni = (int)gr.in_place.size(), no = (int)gr.out_place.size();
    for (int k = 0; k < ni; ++k) {
      in[k] = where(gr.in_place[k]);
      if (!in[k]) return set_err(ctx, DISC_ERR_INVALID_ARG, "null input pointer");
    }
    for (int k = 0; k < no; ++k) {
      outp[k] = where(gr.out_place[k]);
      if (!outp[k]) return set_err(ctx, DISC_ERR_INVALID_ARG, "null output pointer");
    }
    const int ns = ctx->patterns[gr.pattern_id]->an.n_sym;
    rc = disc_launch(ctx, gr.pattern_id, dims, ns, in, ni, outp, no, ws ? ws + pws : nullptr, total - pws, hip_stream);
    if (rc) return rc;
  }
  return DISC_OK;
  DISC_CATCH(ctx)
}
