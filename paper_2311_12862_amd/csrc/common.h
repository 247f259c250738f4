// Shared declarations of the library's translation units (host side).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <map>
#include <memory>
#include <vector>

#include "spconv.h"

namespace spc {

constexpr int kMaxSplit = 4;
constexpr int kRowPad = 256;  // map rows are padded to a multiple of the largest tile_m
constexpr int kWave = 64;
constexpr int kPlanSlabs = 1;      // plan flags: sort keys start with a spatial slab
constexpr int kPlanOwnOrder = 2;  // and: the library's own order (order.hip) instead of the plain bitmask's (one part)

int hip_fail(hipError_t e, const char* what, const char* file, int line);
#define SPC_HIP(expr)                                                        \
  do {                                                                       \
    hipError_t e__ = (expr);                                                 \
    if (e__ != hipSuccess) return ::spc::hip_fail(e__, #expr, __FILE__, __LINE__); \
  } while (0)
#define SPC_TRY(expr)               \
  do {                              \
    int s__ = (expr);               \
    if (s__ != SPCONV_OK) return s__; \
  } while (0)
#define SPC_LAUNCH_CHECK() SPC_HIP(hipGetLastError())

bool capturing(hipStream_t st);
void* dev_alloc(size_t bytes);
void dev_free(void* p);
// Names the stream that the pool's requests and returns of this thread belong to.
class StreamScope {
 public:
  explicit StreamScope(hipStream_t st);
  ~StreamScope();
  StreamScope(const StreamScope&) = delete;
  StreamScope& operator=(const StreamScope&) = delete;

 private:
  hipStream_t saved_;
};

// Owning device buffer (grow-only when used as scratch).
struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
  DevBuf() = default;
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
  ~DevBuf() { release(); }
  void release() {
    if (p) dev_free(p);
    p = nullptr;
    bytes = 0;
  }
  int alloc(size_t n) {  // exact size, contents undefined
    release();
    if (n == 0) n = 16;
    p = dev_alloc(n);
    if (!p) return SPCONV_ENOMEM;
    bytes = n;
    return SPCONV_OK;
  }
  int reserve(size_t n) { return (n <= bytes && p) ? SPCONV_OK : alloc(n); }
  template <typename T> T* as() const { return reinterpret_cast<T*>(p); }
};

inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Plan of the implicit-GEMM kernels for one side of the map (output rows for
// fwd, input rows for dgrad) and one split count.  Its masks are those of 16-row blocks (the lock-step unit); kernels with
// taller tiles combine them, so one plan serves every kernel.
struct IgemmPlan {
  int n_split = 0;  // 0 = unsorted
  int parts = 1;  // max(1, n_split)
  int64_t rows = 0, rows_pad = 0, n_tiles = 0;
  int lo[kMaxSplit] = {0}, width[kMaxSplit] = {0};
  size_t map_off[kMaxSplit] = {0};  // element offsets into maps
  DevBuf maps;      // reordered maps, part i: int32 [rows_pad][width[i]]  (unused when n_split == 0)
  DevBuf perm;      // int32 [parts][rows_pad]                              (unused when n_split == 0)
  DevBuf tilemask;  // uint32 [parts][n_tiles]: masks of 16-row blocks, bits relative to lo[i]  (unused when n_split == 0)
  bool slabs = false;  // sort keys start with a spatial slab: contiguous ranges of the order are spatially compact
};

// Weight-stationary view of the map: the present pairs of each offset, compacted in row order (the M_delta of Section
// 2.2.1).  Made once per kmap, by the first wgrad or fetch-on-demand call.
struct PairList {
  DevBuf pairs;           // int2 [cap]: (output row n, input row j), offset-major
  int64_t cap = 0;        // n_pairs, or the bound n_out * V while an asynchronous build is pending
  DevBuf seg;             // int32 [V+1]: pairs of offset k are seg[k]..seg[k+1]
};

struct PairItem {
  int32_t k, pair_begin, pair_end, pad;  // pairs [pair_begin, pair_end) of offset k
};

// The pair list cut into work items of about `target` pairs of one offset each (fetch-on-demand).
struct ItemPlan {
  int64_t target = 0;
  int max_items = 0;  // launch bound: V + ceil(pairs / target)
  DevBuf items;       // PairItem [max_items]
  DevBuf item_seg;    // int32 [V+2]: items of offset k are item_seg[k]..item_seg[k+1]; [V+1] = n_items
};

struct SideMap {      // one output-stationary table: rows x V
  int64_t rows = 0, rows_pad = 0;
  DevBuf map;         // int32 [rows_pad][V]
  DevBuf mask;        // uint32 [rows_pad]
  // The input side of a stride-2 build over the box: int32 [n_in][8] (K = 2: [n_in][1]), the outputs that each input row has an offset
  // to, -1 where there is none; the side is made from them without a search, and they go when it is there.  Empty where they would be
  // more than the output side is.
  DevBuf cands;
  bool ready = false;
  std::map<std::pair<int, int>, std::unique_ptr<IgemmPlan>> plans;  // (n_split, flags)
};

}  // namespace spc

struct spconv_kmap {
  int K = 3, V = 27, stride = 1, transposed = 0;
  int dilated = 0;  // stride 1 with P_out = every point that has an input in its neighbourhood (not P_in)
  int64_t n_in = 0, n_out = 0, n_pairs = -1;
  hipStream_t build_stream = nullptr;
  hipStream_t last_stream = nullptr;  // stream of the most recent call that used this kmap
  // coordinate sets, reference-counted like the tables (a transposed partner holds the same two)
  std::shared_ptr<spc::DevBuf> in_coords_ref, out_coords_ref;
  spc::DevBuf& in_coords;
  spc::DevBuf& out_coords;
  // The two tables are reference-counted: a kmap and the kmap of its paired transposed
  // convolution hold the same two tables with the roles exchanged (spconv_kmap_transpose).
  std::shared_ptr<spc::SideMap> out_ref, in_ref;
  spc::SideMap& out_side;  // M: rows = n_out, entries index input rows
  spc::SideMap& in_side;   // T: rows = n_in, T[j][k] = n  <=>  M[n][k] = j (built on demand)
  spconv_kmap()
      : in_coords_ref(std::make_shared<spc::DevBuf>()), out_coords_ref(std::make_shared<spc::DevBuf>()),
        in_coords(*in_coords_ref), out_coords(*out_coords_ref), out_ref(std::make_shared<spc::SideMap>()),
        in_ref(std::make_shared<spc::SideMap>()), out_side(*out_ref), in_side(*in_ref) {}
  spconv_kmap(std::shared_ptr<spc::SideMap> out_table, std::shared_ptr<spc::SideMap> in_table,
              std::shared_ptr<spc::DevBuf> in_rows, std::shared_ptr<spc::DevBuf> out_rows)
      : in_coords_ref(std::move(in_rows)), out_coords_ref(std::move(out_rows)), in_coords(*in_coords_ref),
        out_coords(*out_coords_ref), out_ref(std::move(out_table)), in_ref(std::move(in_table)), out_side(*out_ref),
        in_side(*in_ref) {}
  spconv_kmap(const spconv_kmap&) = delete;
  spconv_kmap& operator=(const spconv_kmap&) = delete;
  std::unique_ptr<spc::PairList> pair_list;
  // The pair count that decides between the pairs and the map (wgrad_from_map): n_pairs as the first call that chose by itself
  // knew it, -1 where a build was still pending.  It stays, so that what becomes known later does not give the same call another
  // kernel, other bits and another workspace.
  static constexpr int64_t kNotAsked = -2;
  int64_t wgrad_known_pairs = kNotAsked;
  std::map<int64_t, std::unique_ptr<spc::ItemPlan>> item_plans;  // by target
  // K = 5 (125 offsets): the kmap is held as its five x-planes, each a submanifold map of 25 offsets
  // (dx = g - 2) over the same rows, so that masks, sort keys and tile masks stay 32-bit words and
  // every kernel runs on a plane as it runs on a 27-offset map; the planes' results are summed like
  // the parts of a split.  Offset k of the whole map is offset k % 25 of plane k / 25.
  std::vector<std::unique_ptr<spconv_kmap>> groups;
  spc::DevBuf scratch;    // split partial sums / wgrad partial tiles
  // build whose status was not read yet: the pinned block the probe kernel publishes flags and
  // pair count to, with the event that marks the probe's completion
  void* pending_host = nullptr;
  bool pending = false;
  int build_status = SPCONV_OK;  // verdict of the build once resolved: every later spconv_kmap_status returns it
  ~spconv_kmap();
  bool submanifold() const { return stride == 1 && !transposed && !dilated; }
};

namespace spc {

// ---- kmap.hip
int kmap_build(const int32_t* coords, int64_t N, int K, int stride, int transposed, bool async, hipStream_t st,
               spconv_kmap** out, bool dilate = false);
int kmap_status(spconv_kmap* km, hipStream_t st);  // resolves a pending asynchronous build (synchronises)
int kmap_build_in_side(spconv_kmap* km, hipStream_t st);
int kmap_count_pairs(spconv_kmap* km, hipStream_t st, int64_t* per_k /*[V] or null*/);
int kmap_export_mask_words(const spconv_kmap* km, uint32_t* dst, hipStream_t st);  // K = 5: [n_out][4]
int kmap_transpose(spconv_kmap* src, hipStream_t st, spconv_kmap** out);
int kmap_pointwise(spconv_kmap* src, int on_outputs, hipStream_t st, spconv_kmap** out);

// ---- sort.hip
// Stable LSD radix sort of n (key, value) pairs on key bits [0, key_bits).
// keys/vals are ping-pong buffers of n elements each; *in_b tells where the
// result ended up (0: buffer a, 1: buffer b).  hist must hold
// sort_hist_elems(n) uint32.
size_t sort_hist_elems(int64_t n);
// plan.hip: one launch per digit, at most 393216 keys (SPCONV_EINVAL beyond); see there for error_word
int msort_keys_u32(uint32_t* key_a, uint32_t* key_b, int64_t n, int key_bits, unsigned* error_word, unsigned error_bit,
                   hipStream_t st, int* in_b);
// Exclusive scan in place; `sums` is scratch of scan_sums_elems(elems) counters.
size_t scan_sums_elems(int64_t elems);
int scan_u32_inplace(uint32_t* data, int64_t elems, uint32_t* sums, hipStream_t st);
int radix_sort_u32(uint32_t* key_a, uint32_t* key_b, int32_t* val_a, int32_t* val_b, int64_t n,
                   int key_bits, uint32_t* hist, hipStream_t st, int* in_b);
// Keys only, 64-bit, on the digit positions whose bits are set in `varying`.
int radix_sort_u64(uint64_t* key_a, uint64_t* key_b, int64_t n, uint64_t varying, uint32_t* hist,
                   hipStream_t st, int* in_b);

// ---- launch arithmetic.  Everything a launch derives from the layer's shape is computed by these
// host functions and by nothing else (the run functions call them), so that it can be checked on
// the CPU: spconv_describe_launch reports it, and a test walks the index formulas of the kernels
// over a grid of shapes.  They return SPCONV_EINVAL for shapes the kernels do not take.
struct PlanShape {  // plan_get: parts of the offset range, padded rows, tiles
  int parts = 1;
  int lo[kMaxSplit] = {0}, width[kMaxSplit] = {0};
  size_t map_off[kMaxSplit] = {0};  // element offsets of the parts' reordered maps
  size_t map_elems = 0;             // all parts together
  int64_t rows_pad = 0, n_tiles = 0;
};
int plan_shape(int V, int64_t rows, int n_split, int tile_m, PlanShape* s);

struct WaveShape {  // igemm_wave_run (kernel 1)
  int bn = 0, waves = 0, ks = 0, pack = 1, max_width = 0, threads = 0;  // pack: offsets that share a matrix instruction
  int slab_bytes = 0, map_bytes = 0, weight_bytes = 0;
  size_t lds_bytes = 0;
  unsigned grid[3] = {0, 0, 0};
  unsigned feats_bytes = 0;
};
int igemm_wave_shape(int V, int n_split, int64_t rows, int64_t rows_src, int c_red, int c_out, int tile_n,
                     WaveShape* s);

int igemm_wave_planes_shape(int64_t rows, int64_t rows_src, int c_red, int c_out, WaveShape* s);  // K = 5 in one launch

struct TileShape {  // igemm_run (kernel 2 and the fp32 kernel)
  int bm = 0, bn = 0, kc = 0, nw = 0, threads = 0;
  size_t lds_bytes = 0;
  unsigned grid[3] = {0, 0, 0};
  unsigned feats_bytes = 0;
};
int igemm_tile_shape(int V, int n_split, int64_t rows, int64_t rows_src, int c_red, int c_out, int tile_m, int tile_n,
                     bool f32, bool dgrad, TileShape* s);

struct RingShape {  // igemm_ring_run (tiles loaded straight into LDS; every fp32 layer)
  int bm = 0, bn = 0, nwk = 0, nwr = 0, piece = 0;  // rows and columns of a workgroup, K groups, tiles (one below the other), bytes of a row per unit
  int threads = 0, n_cols = 0;
  int64_t n_tiles = 0;
  size_t lds_bytes = 0;
  unsigned grid[3] = {0, 0, 0};
  unsigned feats_bytes = 0;
};
// small_tiles: 32-row tiles, and column tiles of fp32 that the layer's width does not ask for, may be chosen
int igemm_ring_shape(int V, int n_split, int64_t rows, int64_t rows_src, int c_red, int c_out, bool f32, bool dgrad,
                     bool small_tiles, RingShape* s);

// ---- plan.hip
// flags: kPlanSlabs, kPlanOwnOrder (each combination is a plan of its own in the cache)
int plan_get(spconv_kmap* km, SideMap& side, int n_split, int flags, hipStream_t st, IgemmPlan** out);
int plan_mac_units(spconv_kmap* km, SideMap& side, IgemmPlan* plan, int group_rows, hipStream_t st,
                   int64_t* executed);
int pair_list_get(spconv_kmap* km, hipStream_t st, PairList** out);
int item_plan_get(spconv_kmap* km, int64_t target, hipStream_t st, ItemPlan** out);

// ---- order.hip: fills perm, maps and tilemask of a one-part plan in the library's own order
int order_rows(const SideMap& side, int V, IgemmPlan& p, hipStream_t st);

// ---- igemm.hip
struct IgemmArgs {
  const void* feats;    // [rows_src][c_red]
  const void* weights;  // [V][C_in][C_out] (always the forward layout)
  void* out;            // [rows][c_out_eff] in dtype, or nullptr when partial sums are used
  float* partial;       // [parts][rows][c_out_eff] fp32: the kernels write partial sums whenever this is set
  int C_in, C_out;      // of the layer (forward orientation)
  int dgrad;            // 0: reduce over C_in, produce C_out.  1: reduce over C_out, produce C_in
  int mirror;           // weight slice of map column k is V-1-k (dgrad on the submanifold map itself)
  spconv_dtype dtype;
  int tile_n;           // 0 = auto
};
int igemm_run(const spconv_kmap* km, const SideMap& side, const IgemmPlan& plan, const IgemmArgs& a, int tile_m,
              hipStream_t st);
// ---- igemm_ring.hip
int igemm_ring_run(const spconv_kmap* km, const SideMap& side, const IgemmPlan& plan, const IgemmArgs& a, const RingShape& s,
                   hipStream_t st);
// ---- igemm_wave.hip (weights resident in LDS)
int igemm_wave_pick_bn(int V, int n_split, int c_red, int c_out, int tile_n, int* waves_out);
int igemm_wave_run(const spconv_kmap* km, const SideMap& side, const IgemmPlan& plan, const IgemmArgs& a,
                   hipStream_t st);
int igemm_wave_planes_run(const spconv_kmap* km, const IgemmArgs& a, hipStream_t st);  // km: K = 5, map order
int split_reduce(const float* partial, int parts, int64_t rows, int c, spconv_dtype dtype, void* out,
                 hipStream_t st);

// ---- fod.hip (fetch-on-demand dataflow; wp must have been cut into items of tile_m pairs)
bool fod_supported(const spconv_kmap* km, int dgrad, int C_in, int C_out, spconv_dtype dtype);
int fod_run(spconv_kmap* km, const ItemPlan& wp, const IgemmArgs& a, int tile_m, void* dst, hipStream_t st);

// ---- wgrad.hip
int64_t wgrad_auto_pairs(const spconv_kmap* km, int C_in, int C_out, spconv_dtype dtype);
bool wgrad_from_map(const spconv_kmap* km, int C_in, int C_out, spconv_dtype dtype);
int wgrad_map_run(spconv_kmap* km, const void* feats, const void* dout, int C_in, int C_out, spconv_dtype dtype, float* dweights, hipStream_t st);
int wgrad_run(spconv_kmap* km, const PairList& pl, int64_t piece_pairs, const void* feats, const void* dout, int C_in, int C_out,
              spconv_dtype dtype, float* dweights, hipStream_t st);

}  // namespace spc
