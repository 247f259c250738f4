// Kernel-map construction: coordinate hash table, output-coordinate
// generation for strided maps, neighbour probe, neighbour bitmask, and the
// input-side (transposed) table that dgrad of strided maps walks.
//
// The paper counts these mapping operations as a cost centre (Sections 4.2,
// 6.1, 6.3) but gives no algorithm for them; the design below is this
// library's own.  Submanifold 3x3x3 maps, the common case, deal their rows into buckets
// of neighbouring blocks, each of which one workgroup hashes into LDS and looks up there;
// 5x5x5 maps hash runs of four cells along z into a table in memory.  The other maps use one 16-byte
// slot per key (64-bit packed coordinate + row index) in an open-addressing
// table at load factor <= 0.5 and one probe lane per (output row, offset), so
// that map writes are contiguous per wave and the bitmask comes from a wave
// ballot; stride-2 maps are built over a bit per cell of the coarse points'
// box; K = 5 maps are held as five planes of 25 offsets.
#include "common.h"

#include <atomic>
#include <chrono>
#include <thread>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

namespace spc {
namespace {

constexpr unsigned long long kEmpty = ~0ull;

// SORT: a sort's bounded wait ran out; BOX: the coarse points' bounding box is too large for a bit per cell
enum : unsigned long long { FLAG_RANGE = 1, FLAG_DUP = 2, FLAG_FULL = 4, FLAG_SORT = 8, FLAG_BOX = 16 };
constexpr int kRetryGeneralSort = 1;  // (internal) build again with the general sort
constexpr int kRetryTable = 2;        // (internal) build with a hash table (of the coarse points, or of a submanifold map's rows)

// Control block read back by the host at the build's synchronisation point.  The pair counter
// is spread over 64 cache lines (one atomic per probe workgroup) so that the adds do not queue
// up on one address.
constexpr int kPairSlots = 64;
constexpr int kPlaneSlots = 12;  // K = 5: pair-count slots per plane (5 x 12 <= kPairSlots)
struct Ctl {
  unsigned long long flags, count, pad[14];
  unsigned long long pairs[kPairSlots * 16];
  unsigned long long key_or[kPairSlots * 16], key_and[kPairSlots * 16];  // spread like pairs
  unsigned long long entries[kPairSlots * 16];  // present map entries, counted from the finished map
  unsigned tick_top, pad2[15];     // pair slots whose workgroups have all arrived
};

// What a submanifold build hands to the host: written by the probe straight into pinned host
// memory, so that no copy has to be enqueued behind the build.
// What an asynchronous build leaves in pinned host memory, in one 8-byte word so that one store
// publishes it: bit 63 = written, bits 48..55 = error flags, bits 0..47 = pair count.
// Whoever waits polls all that the kernels given the block store last, each of them once, and then hands it to the next build.
struct HostResult {
  unsigned long long word;
  unsigned long long outputs;  // with bit 63 like word (kPublishOutputs)
  // what builds over hash tables hand over (kPublishAll): written before `ready`
  unsigned long long flags, count, key_or, key_and, pairs, entries, plane_pairs[5];
  unsigned long long ready;
};
constexpr unsigned long long kHostReady = 1ull << 63;

__device__ __forceinline__ bool coord_ok(int b, int x, int y, int z) {
  return (unsigned)b <= 65534u && (unsigned)(x + 32768) <= 65535u && (unsigned)(y + 32768) <= 65535u &&
         (unsigned)(z + 32768) <= 65535u;
}

// (b, x, y, z) -> 64-bit key whose unsigned order is the lexicographic order of (b, x, y, z).
__device__ __forceinline__ unsigned long long pack_key(int b, int x, int y, int z) {
  return ((unsigned long long)(unsigned)b << 48) | ((unsigned long long)(unsigned)(x + 32768) << 32) |
         ((unsigned long long)(unsigned)(y + 32768) << 16) | (unsigned long long)(unsigned)(z + 32768);
}

// The table is an array of buckets of four 16-byte slots (one 64-byte line).  A key hashes to a
// bucket; insertion takes the first free slot of the bucket, in order, and moves on to the next
// bucket when all four are taken.  A lookup reads one line per step (four loads in flight) and
// stops at the first empty slot; at load <= 0.5 a second step is rare.
__device__ __forceinline__ unsigned hash_bucket(unsigned long long key, int log_cap) {
  return (unsigned)((key * 0x9E3779B97F4A7C15ull) >> (64 - (log_cap - 2)));
}

// 0: inserted, 1: key already there, 2: table full (cannot happen at load <= 0.5)
__device__ __forceinline__ int table_insert(unsigned long long* tab, int log_cap, unsigned long long key,
                                            int val, unsigned* slot_out) {
  const unsigned bucket_mask = (1u << (log_cap - 2)) - 1u;
  unsigned b = hash_bucket(key, log_cap);
  for (unsigned it = 0; it <= bucket_mask; ++it) {
    for (unsigned i = 0; i < 4; ++i) {
      const unsigned s = b * 4 + i;
      const unsigned long long old = atomicCAS(&tab[2 * (size_t)s], kEmpty, key);
      if (old == kEmpty) {
        tab[2 * (size_t)s + 1] = (unsigned long long)(unsigned)val;
        if (slot_out) *slot_out = s;
        return 0;
      }
      if (old == key) {
        if (slot_out) *slot_out = s;
        return 1;
      }
    }
    b = (b + 1) & bucket_mask;
  }
  return 2;
}

__device__ __forceinline__ int table_find(const unsigned long long* tab, int log_cap, unsigned long long key,
                                          unsigned* slot_out) {
  const unsigned bucket_mask = (1u << (log_cap - 2)) - 1u;
  unsigned b = hash_bucket(key, log_cap);
  for (unsigned it = 0; it <= bucket_mask; ++it) {
    const ulonglong2* line = reinterpret_cast<const ulonglong2*>(tab) + (size_t)b * 4;
    const ulonglong2 e0 = line[0], e1 = line[1], e2 = line[2], e3 = line[3];  // four loads in flight
    if (e0.x == key) {
      if (slot_out) *slot_out = b * 4;
      return (int)(unsigned)e0.y;
    }
    if (e0.x == kEmpty) return -1;
    if (e1.x == key) {
      if (slot_out) *slot_out = b * 4 + 1;
      return (int)(unsigned)e1.y;
    }
    if (e1.x == kEmpty) return -1;
    if (e2.x == key) {
      if (slot_out) *slot_out = b * 4 + 2;
      return (int)(unsigned)e2.y;
    }
    if (e2.x == kEmpty) return -1;
    if (e3.x == key) {
      if (slot_out) *slot_out = b * 4 + 3;
      return (int)(unsigned)e3.y;
    }
    if (e3.x == kEmpty) return -1;
    b = (b + 1) & bucket_mask;
  }
  return -1;
}

__device__ __forceinline__ int floor_div(int a, int s) {
  int q = a / s;
  return (a % s != 0 && a < 0) ? q - 1 : q;
}

// Insert key(p_j) -> j for every input row; flags range and duplicate errors.
__global__ void __launch_bounds__(256) k_insert_rows(const int4* __restrict__ coords, int n,
                                                     unsigned long long* tab, int log_cap, Ctl* ctl,
                                                     int4* __restrict__ keep) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int4 c = coords[j];
  keep[j] = c;  // the kmap's own copy of the caller's rows
  if (!coord_ok(c.x, c.y, c.z, c.w)) {
    atomicOr(&ctl->flags, FLAG_RANGE);
    return;
  }
  const int r = table_insert(tab, log_cap, pack_key(c.x, c.y, c.z, c.w), j, nullptr);
  if (r == 1) atomicOr(&ctl->flags, FLAG_DUP);
  if (r == 2) atomicOr(&ctl->flags, FLAG_FULL);
}

// Coarse coordinates floor(p / s): de-duplicate through a second table, append each
// new key to ukeys (order arbitrary; sorted afterwards), and reduce OR / AND of the
// keys so that the host knows which key bytes vary.  Every thread of a workgroup; live: it has a row.
template <int WAVES = 4>  // of the workgroup
__device__ __forceinline__ void coarse_unique(bool live, int4 c, int stride, unsigned long long* tab, int log_cap,
                                              unsigned long long* __restrict__ ukeys, Ctl* ctl) {
  __shared__ unsigned long long s_or[WAVES], s_and[WAVES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bool fresh = false;
  unsigned long long key = 0, k_or = 0, k_and = ~0ull;
  if (live) {
    if (!coord_ok(c.x, c.y, c.z, c.w)) atomicOr(&ctl->flags, FLAG_RANGE);
    if (coord_ok(c.x, c.y, c.z, c.w)) {
      key = pack_key(c.x, floor_div(c.y, stride), floor_div(c.z, stride), floor_div(c.w, stride));
      const int r = table_insert(tab, log_cap, key, 0, nullptr);
      fresh = (r == 0);
      if (r == 2) atomicOr(&ctl->flags, FLAG_FULL);
      k_or = key;
      k_and = key;
    }
  }
  // workgroup-aggregated append: one counter atomic per workgroup, ranks from ballots
  __shared__ unsigned wave_cnt[WAVES];
  __shared__ unsigned long long block_base;
  const unsigned long long bal = __ballot(fresh);
  if (lane == 0) wave_cnt[wave] = (unsigned)__popcll(bal);
  for (int o = 32; o > 0; o >>= 1) {
    k_or |= __shfl_xor(k_or, o);
    k_and &= __shfl_xor(k_and, o);
  }
  if (lane == 0) {
    s_or[wave] = k_or;
    s_and[wave] = k_and;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned total = 0;
    unsigned long long all_or = 0, all_and = ~0ull;
    for (int w = 0; w < WAVES; ++w) total += wave_cnt[w], all_or |= s_or[w], all_and &= s_and[w];
    block_base = total ? atomicAdd(&ctl->count, (unsigned long long)total) : 0ull;
    const int slot = (blockIdx.x % kPairSlots) * 16;
    atomicOr(&ctl->key_or[slot], all_or);
    atomicAnd(&ctl->key_and[slot], all_and);
  }
  __syncthreads();
  if (fresh) {
    unsigned before = 0;
    for (int w = 0; w < wave; ++w) before += wave_cnt[w];
    ukeys[block_base + before + __popcll(bal & ((1ull << lane) - 1ull))] = key;
  }
}

__global__ void __launch_bounds__(256) k_coarse_unique(const int4* __restrict__ coords, int n, int stride,
                                                       unsigned long long* tab, int log_cap,
                                                       unsigned long long* __restrict__ ukeys, Ctl* ctl,
                                                       int4* __restrict__ keep) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  int4 c = make_int4(-1, 0, 0, 0);
  if (j < n) {
    c = coords[j];
    if (keep) keep[j] = c;  // the kmap's own copy of the caller's rows (builds without a fine table)
  }
  coarse_unique(j < n, c, stride, tab, log_cap, ukeys, ctl);
}

// Candidate outputs of a dilated stride-1 map: q = p - delta for every input p and offset delta
// (Equation 1 with P_out = every point that reads at least one input), de-duplicated and appended
// like the coarse points above.  One thread per (input row, offset).
template <int K>
__global__ void __launch_bounds__(256) k_dilate_unique(const int4* __restrict__ coords, long long n,
                                                       unsigned long long* tab, int log_cap,
                                                       unsigned long long* __restrict__ ukeys, Ctl* ctl) {
  constexpr int V = K * K * K, R = (K - 1) / 2;
  __shared__ unsigned long long s_or[4], s_and[4];
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long j = t / V;
  const int k = (int)(t - j * V);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bool fresh = false;
  unsigned long long key = 0, k_or = 0, k_and = ~0ull;
  if (j < n) {
    const int4 c = coords[j];
    const int qx = c.y - (k / (K * K) - R), qy = c.z - ((k / K) % K - R), qz = c.w - (k % K - R);
    if (coord_ok(c.x, c.y, c.z, c.w)) {  // (an invalid input row is flagged by the insert kernel)
      if (!coord_ok(c.x, qx, qy, qz)) {
        atomicOr(&ctl->flags, FLAG_RANGE);  // an output beside the packable range
      } else {
        key = pack_key(c.x, qx, qy, qz);
        const int r = table_insert(tab, log_cap, key, 0, nullptr);
        fresh = (r == 0);
        if (r == 2) atomicOr(&ctl->flags, FLAG_FULL);
        k_or = key;
        k_and = key;
      }
    }
  }
  __shared__ unsigned wave_cnt[4];
  __shared__ unsigned long long block_base;
  const unsigned long long bal = __ballot(fresh);
  if (lane == 0) wave_cnt[wave] = (unsigned)__popcll(bal);
  for (int o = 32; o > 0; o >>= 1) {
    k_or |= __shfl_xor(k_or, o);
    k_and &= __shfl_xor(k_and, o);
  }
  if (lane == 0) {
    s_or[wave] = k_or;
    s_and[wave] = k_and;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned total = wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
    block_base = total ? atomicAdd(&ctl->count, (unsigned long long)total) : 0ull;
    const int slot = (blockIdx.x % kPairSlots) * 16;
    atomicOr(&ctl->key_or[slot], s_or[0] | s_or[1] | s_or[2] | s_or[3]);
    atomicAnd(&ctl->key_and[slot], s_and[0] & s_and[1] & s_and[2] & s_and[3]);
  }
  __syncthreads();
  if (fresh) {
    unsigned before = 0;
    for (int w = 0; w < wave; ++w) before += wave_cnt[w];
    ukeys[block_base + before + __popcll(bal & ((1ull << lane) - 1ull))] = key;
  }
}

__global__ void __launch_bounds__(256) k_decode_keys(const unsigned long long* __restrict__ keys, int n,
                                                     int4* __restrict__ coords) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const unsigned long long k = keys[i];
  int4 c;
  c.x = (int)(k >> 48);
  c.y = (int)((k >> 32) & 0xFFFF) - 32768;
  c.z = (int)((k >> 16) & 0xFFFF) - 32768;
  c.w = (int)(k & 0xFFFF) - 32768;
  coords[i] = c;
}

// After sorting the unique coarse keys: store each key's rank as its table value.
__global__ void __launch_bounds__(256) k_assign_rank(const unsigned long long* __restrict__ keys, int n,
                                                     unsigned long long* tab, int log_cap) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  unsigned slot = 0;
  if (table_find(tab, log_cap, keys[i], &slot) >= 0) tab[2 * (size_t)slot + 1] = (unsigned long long)(unsigned)i;
}

// One lane per (row, offset).  A wave covers 64 / V rows, so that its V-lane
// groups write contiguous map entries and a single ballot yields the bitmasks.
//   TRANSPOSED = false: row coords are output points q; look up s*q + delta.
//   TRANSPOSED = true : row coords are fine points f; look up (f - delta) / s if divisible.
template <int K, bool TRANSPOSED>
__global__ void __launch_bounds__(256) k_probe(const int4* __restrict__ rows, int n_rows, int stride,
                                               const unsigned long long* __restrict__ tab, int log_cap,
                                               int* __restrict__ map, unsigned* __restrict__ mask, Ctl* ctl) {
  __shared__ unsigned wave_pairs[4];
  constexpr int V = K * K * K;
  constexpr int RPW = 64 / V;
  constexpr int R = (K - 1) / 2;
  const int lane = threadIdx.x & 63;
  const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int sub = lane / V, k = lane - sub * V;
  const long long row = wave * RPW + sub;
  const bool active = (sub < RPW) && (row < n_rows);
  int found = -1;
  if (active) {
    const int4 c = rows[row];
    const int dx = k / (K * K) - R, dy = (k / K) % K - R, dz = k % K - R;
    int tx, ty, tz;
    bool ok = true;
    if (!TRANSPOSED) {
      tx = stride * c.y + dx;
      ty = stride * c.z + dy;
      tz = stride * c.w + dz;
    } else {
      const int fx = c.y - dx, fy = c.z - dy, fz = c.w - dz;
      tx = floor_div(fx, stride);
      ty = floor_div(fy, stride);
      tz = floor_div(fz, stride);
      ok = (tx * stride == fx) && (ty * stride == fy) && (tz * stride == fz);
    }
    if (ok && coord_ok(c.x, tx, ty, tz)) found = table_find(tab, log_cap, pack_key(c.x, tx, ty, tz), nullptr);
    map[row * V + k] = found;
  }
  const unsigned long long bal = __ballot(found >= 0);
  if (active && k == 0) mask[row] = (unsigned)((bal >> (sub * V)) & ((1ull << V) - 1ull));
  // number of present pairs: one atomic per workgroup
  if (lane == 0) wave_pairs[threadIdx.x >> 6] = (unsigned)__popcll(bal);
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned n = wave_pairs[0] + wave_pairs[1] + wave_pairs[2] + wave_pairs[3];
    if (n) atomicAdd(&ctl->pairs[(blockIdx.x % kPairSlots) * 16], (unsigned long long)n);
  }
}

// Strided 3x3x3 map built from the input side.  Input p meets output q exactly when
// p = s*q + delta with delta in {-1, 0, 1}^3 (Eq. 1 with stride s), so per axis q is floor(p/s)
// (delta = p - s*q, if that is <= 1) or floor(p/s) + 1 (delta = p - s*q, if that is >= -1): at most
// 2x2x2 candidates, tried by 8 lanes per input row, each one lookup of q's rank in the table of
// coarse points.  At stride 2 that is 3.4 lookups per input on average, against 27 per output when
// probing from the output side.  The map was preset to -1; the masks are derived from it
// afterwards.  Plain stores: duplicate input rows write one entry twice, which shows as fewer
// present entries in the finished map than hits counted here.
__global__ void __launch_bounds__(256)
    k_scatter_down3(const int4* __restrict__ rows, int n_rows, int stride, const unsigned long long* __restrict__ tab,
                    int log_cap, int* __restrict__ map, Ctl* ctl) {
  __shared__ unsigned wave_pairs[4];
  constexpr int V = 27;
  const int lane = threadIdx.x & 63;
  const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const long long row = wave * 8 + (lane >> 3);
  const int cand = lane & 7;
  bool found = false;
  if (row < n_rows) {
    const int4 c = rows[row];
    if (coord_ok(c.x, c.y, c.z, c.w)) {
      const int pc[3] = {c.y, c.z, c.w};
      int q[3], d[3];
      bool ok = true;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int up = (cand >> (2 - a)) & 1;
        q[a] = floor_div(pc[a], stride) + up;
        d[a] = pc[a] - stride * q[a];
        ok = ok && d[a] >= -1 && d[a] <= 1;
      }
      if (ok && coord_ok(c.x, q[0], q[1], q[2])) {
        const int n = table_find(tab, log_cap, pack_key(c.x, q[0], q[1], q[2]), nullptr);
        if (n >= 0) {
          const int k = ((d[0] + 1) * 3 + (d[1] + 1)) * 3 + (d[2] + 1);
          map[(long long)n * V + k] = (int)row;
          found = true;
        }
      }
    }
  }
  const unsigned long long bal = __ballot(found);
  if (lane == 0) wave_pairs[threadIdx.x >> 6] = (unsigned)__popcll(bal);
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned n = wave_pairs[0] + wave_pairs[1] + wave_pairs[2] + wave_pairs[3];
    if (n) atomicAdd(&ctl->pairs[(blockIdx.x % kPairSlots) * 16], (unsigned long long)n);
  }
}

// ---- stride-2 builds over a bit per cell ----
// The coarse points floor(p / 2) of a scan fill a box of a few hundred cells per row.  One bit per cell, set by the rows, is the
// de-duplication, the lexicographic sort (the order of the bits) and the look-up table (a point's row is the number of set
// bits before its own: a prefix per 32 cells and a population count) at once; nothing is hashed, sorted or probed, and the
// host waits once, at the end.  The cells are cut into groups of equal length, and the groups dealt out to as many chunks as there are
// workgroups, neighbouring groups to different ones (group_at).  The rows are dealt to the chunks of their coarse
// points, and one workgroup per chunk sets its bits in LDS and writes them with their prefixes: nothing is cleared beforehand and no
// atomic leaves the CU.  Launches: the box, dealing, bits, group prefixes (and the presets of
// the map), the map from the input side (and the coordinates), masks.  Whole waited 3x3x3 builds with bits in memory (cleared, marked by an
// atomic per row, which the memory side takes at 10 per ns, counted) and so, us: LiDAR-like scans of 2k rows 72, 45; 10k 67, 47; 30k 72, 49;
// 100k 90, 60; 200k (127k outputs) 110, 77; 400k 152, 103; a room of 60k 79, 51; 300k 141, 107 (with the copy of shrink_to_outputs).
// De-duplication through a hash table, a radix sort and table look-ups took 1.3 to 2.3 times as long as bits in memory.
// A box of more than kCellsPerRow cells a row (a scan of 5 cm voxels has about 450) is left to the table: the dealing launch
// empties one in the bitmap's place, the launch behind it fills it, and the host, which reads the box's verdict behind that, goes on
// with the sort.  Whole builds of points spread over 60,000 cells an axis, us, all through the table and so: 2k rows 150, 152;
// 20k 218, 219; 100k 253, 255; 200k 290, 289.
constexpr int kBoxBlocks = 256;
constexpr int kCellsPerRow = 2048;
constexpr int64_t kMaxBoxWords = 1ll << 26;
constexpr int kBoxDealers = 256, kBoxDealThreads = 512;  // workgroups of k_box_deal at most: one per thread of k_box_bits
constexpr int kMaxChunks = 2048, kMaxGroups = 32768;
constexpr int kLogLdsWords = 13, kLdsWords = 1 << kLogLdsWords;  // words of a chunk that are in LDS at a time: a window
constexpr int kMaxWindows = 4;     // (a chunk has kMaxBoxWords / kMaxChunks words at most, fewer chunks 400 kCellsPerRow / 32 and a group)
static_assert(kMaxBoxWords / kMaxChunks <= kMaxWindows * kLdsWords && 400 * kCellsPerRow / 32 + kLdsWords / 2 <= kMaxWindows * kLdsWords, "");
constexpr int kBaseThreads = 1024;
static_assert(kMaxBoxWords / kMaxGroups <= kLdsWords && kMaxGroups % (4 * kBaseThreads) == 0 && kMaxChunks % kBaseThreads == 0, "");
constexpr int kBitsThreads = 1024;  // (256: the chunks at a scanner's place, of thousands of rows, took 22 us)

struct Box {
  int lo[4];         // of (b, x, y, z)
  unsigned span[4];  // (up to 65536 each)
  unsigned words;    // of 32 cells; 0: nothing to do
  unsigned shift;    // a group is 2^shift words
  unsigned windows;  // of a chunk (1 except in sparse boxes)
  unsigned flags;
  __host__ __device__ unsigned groups() const { return (words + (1u << shift) - 1u) >> shift; }
};

// Most groups of a box.  A chunk has up to 64, so that rows which crowd into a part of the box are shared among many workgroups all the
// same: with chunks of neighbouring cells, one point far from a plane of 200k rows left nearly all of them to one workgroup.  Whole 3x3x3
// builds without and with such a point, us, so and in groups: a plane of 200k 74, 395 and 72, 96; a room of 60k 51, 105 and 51, 60; scans
// of 100k 62, 98 and 61, 70; 400k 103, 138 and 102, 139 (the cells of the larger box, which are written, are the rest).
// Rows are dealt to the windows of a chunk, so that none is looked at for a window that it is not in, and a crowded window takes its rows
// dealer by dealer: planes of 203k, 400k and 1M rows without a gap, and such a point, with bits in memory, by chunks of neighbouring cells, in
// groups alone, and so, us: 145, 422, 174, 115; 188, 768, 285, 174; 318, 1903, 553, 350.
__host__ __device__ constexpr unsigned most_groups(int chunks) { return chunks * 64 < kMaxGroups ? chunks * 64 : kMaxGroups; }
// Which chunk a group belongs to, and the i-th group of a chunk: every run of `chunks` groups has one of each chunk, and the runs are
// turned against each other, so that cells at any regular distance (a wall along the first axis) do not meet in one chunk.
__device__ __forceinline__ unsigned turn_of(unsigned i, int log_chunks) { return (i * 0x9E3779B1u) >> (32 - log_chunks); }
__device__ __forceinline__ unsigned chunk_of(unsigned group, int log_chunks) {
  return (group + turn_of(group >> log_chunks, log_chunks)) & ((1u << log_chunks) - 1u);
}
__device__ __forceinline__ unsigned group_at(unsigned chunk, unsigned i, int log_chunks) {
  return (i << log_chunks) | ((chunk - turn_of(i, log_chunks)) & ((1u << log_chunks) - 1u));
}

// 32 cells: which are there, and how many are before them in their group.
struct __align__(8) Cells {
  unsigned bits, before;
};

__device__ __forceinline__ unsigned cell_of(const Box& box, int b, int x, int y, int z) {  // (in the box: below 2^31)
  return (((unsigned)(b - box.lo[0]) * box.span[1] + (unsigned)(x - box.lo[1])) * box.span[2] + (unsigned)(y - box.lo[2])) * box.span[3] +
         (unsigned)(z - box.lo[3]);
}

// partial[block] = {least, largest of (b, floor(x / 2), ..), flags} over the rows that the block visits
__global__ void __launch_bounds__(256)
    k_box_bounds(const int4* __restrict__ coords, int n, int4* __restrict__ keep, int* __restrict__ partial) {
  __shared__ int red[4][9];
  int v[9] = {0x7FFFFFFF, 0x7FFFFFFF, 0x7FFFFFFF, 0x7FFFFFFF, (int)0x80000000, (int)0x80000000, (int)0x80000000, (int)0x80000000, 0};
  constexpr int U = 4;
  const int step = gridDim.x * 256;
  for (int r0 = blockIdx.x * 256 + threadIdx.x; r0 < n; r0 += U * step) {
    int4 c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = (long long)r0 + (long long)u * step < n ? coords[r0 + u * step] : make_int4(-1, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if ((long long)r0 + (long long)u * step >= n) continue;
      keep[r0 + u * step] = c[u];
      if (!coord_ok(c[u].x, c[u].y, c[u].z, c[u].w)) {
        v[8] = (int)FLAG_RANGE;
        continue;
      }
      const int q[4] = {c[u].x, c[u].y >> 1, c[u].z >> 1, c[u].w >> 1};
#pragma unroll
      for (int a = 0; a < 4; ++a) v[a] = min(v[a], q[a]), v[4 + a] = max(v[4 + a], q[a]);
    }
  }
#pragma unroll
  for (int a = 0; a < 9; ++a)
    for (int o = 32; o > 0; o >>= 1) {
      const int w = __shfl_xor(v[a], o);
      v[a] = a < 4 ? min(v[a], w) : a < 8 ? max(v[a], w) : v[a] | w;
    }
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int a = 0; a < 9; ++a) red[threadIdx.x >> 6][a] = v[a];
  __syncthreads();
  if (threadIdx.x < 9) {
    const int a = threadIdx.x;
    int w = red[0][a];
    for (int i = 1; i < 4; ++i) w = a < 4 ? min(w, red[i][a]) : a < 8 ? max(w, red[i][a]) : w | red[i][a];
    partial[blockIdx.x * 9 + a] = w;
  }
}

// Every workgroup works out the box; the first one clears the control block, leaves the box for the launches behind, and its flags
// for the host (the word of host).  Workgroup w then deals rows [w per, w per + per): their cells, chunk by chunk, from entries + w per
// on; starts[w][chunk, window] says where each begins.  Where the box is too large, table_slots empty slots of the hash tables take the
// bitmap's place.
__global__ void __launch_bounds__(kBoxDealThreads)
    k_box_deal(const int* __restrict__ partial, int n_partial, long long max_words, const int4* __restrict__ coords, int n, int per,
               int log_chunks, unsigned* __restrict__ entries, unsigned* __restrict__ starts, ulonglong2* __restrict__ table, long long table_slots,
               Box* box_out, Ctl* ctl, HostResult* host) {
  constexpr int U = 2, kWaves = kBoxDealThreads / 64;
  __shared__ int red[4][9];
  __shared__ __align__(16) unsigned place[kMaxChunks * kMaxWindows];  // by chunk and window
  __shared__ unsigned wave_sum[kWaves];
  __shared__ Box s_box;
  const int t = threadIdx.x, lane = t & 63, wib = t >> 6, w = blockIdx.x, chunks = 1 << log_chunks;
  if (t < 256) {
    int v[9];  // (kBoxBlocks == 256 partials at most: one per thread)
#pragma unroll
    for (int a = 0; a < 9; ++a)
      v[a] = t < n_partial ? partial[t * 9 + a] : a < 4 ? 0x7FFFFFFF : a < 8 ? (int)0x80000000 : 0;
#pragma unroll
    for (int a = 0; a < 9; ++a)
      for (int o = 32; o > 0; o >>= 1) {
        const int x = __shfl_xor(v[a], o);
        v[a] = a < 4 ? min(v[a], x) : a < 8 ? max(v[a], x) : v[a] | x;
      }
    if (lane == 0)
#pragma unroll
      for (int a = 0; a < 9; ++a) red[wib][a] = v[a];
  }
  for (int i = t; i < kMaxChunks; i += kBoxDealThreads) place[i] = 0;
  __syncthreads();
  if (t == 0) {
    Box b;
    unsigned long long cells = 1;
    b.flags = 0;
    for (int i = 0; i < 4; ++i) b.flags |= (unsigned)red[i][8];
    for (int a = 0; a < 4; ++a) {
      int lo = red[0][a], hi = red[0][4 + a];
      for (int i = 1; i < 4; ++i) lo = min(lo, red[i][a]), hi = max(hi, red[i][4 + a]);
      b.lo[a] = lo;
      b.span[a] = lo <= hi ? (unsigned)(hi - lo) + 1u : 0u;  // (no valid row: an empty box)
      cells = cells > (1ull << 40) ? cells : cells * b.span[a];
    }
    const unsigned long long words = (cells + 31) / 32;
    if (words > (unsigned long long)max_words) b.flags |= (unsigned)FLAG_BOX;
    b.words = words > (unsigned long long)max_words ? 0u : (unsigned)words;
    // whole fours (k_box_bits writes them), and lines of 16 words where every chunk has one
    b.shift = 2;
    while (b.groups() > (b.shift < 4 ? (unsigned)chunks : most_groups(chunks))) ++b.shift;
    const unsigned most = (b.groups() + chunks - 1) >> log_chunks, in_window = kLdsWords >> b.shift;  // groups of a chunk, of a window
    b.windows = min(max((most + in_window - 1) / in_window, 1u), (unsigned)kMaxWindows);
    s_box = b;
    if (w == 0) {
      *box_out = b;
      __hip_atomic_store(&host->word, kHostReady | ((unsigned long long)b.flags << 48), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  __syncthreads();
  const Box box = s_box;
  if (w == 0) {
    if (t == 0) {
      ctl->flags = box.flags & ~(unsigned)FLAG_BOX;
      ctl->count = 0;
      ctl->tick_top = 0;
    }
    if (t < kPairSlots) {
      ctl->pairs[t * 16] = 0;
      ctl->entries[t * 16] = 0;
      ctl->key_or[t * 16] = 0;
      ctl->key_and[t * 16] = ~0ull;
    }
  }
  if (box.flags & (unsigned)FLAG_BOX) {
    for (long long i = (long long)w * kBoxDealThreads + t; i < table_slots; i += (long long)gridDim.x * kBoxDealThreads)
      table[i] = make_ulonglong2(kEmpty, kEmpty);
    return;
  }
  const int first = (int)min((long long)w * per, (long long)n), last = (int)min((long long)first + per, (long long)n);
  auto visit = [&](auto f) {
    for (long long r0 = first + t; r0 < last; r0 += U * kBoxDealThreads) {
      int4 c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) c[u] = r0 + u * kBoxDealThreads < last ? coords[r0 + u * kBoxDealThreads] : make_int4(-1, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (r0 + u * kBoxDealThreads < last && coord_ok(c[u].x, c[u].y, c[u].z, c[u].w))
          f(cell_of(box, c[u].x, c[u].y >> 1, c[u].z >> 1, c[u].w >> 1));
    }
  };
  const unsigned to_group = 5 + box.shift, to_window = kLogLdsWords - box.shift;
  const int bins = chunks * (int)box.windows;
  auto bin_of = [&](unsigned cell) {
    const unsigned group = cell >> to_group;
    return chunk_of(group, log_chunks) * box.windows + (group >> log_chunks >> to_window);
  };
  if (bins > kMaxChunks) {  // (whole tiles of the sums below)
    for (int i = kMaxChunks + t; i < (bins + kMaxChunks - 1) / kMaxChunks * kMaxChunks; i += kBoxDealThreads) place[i] = 0;
    __syncthreads();
  }
  visit([&](unsigned cell) { atomicAdd(&place[bin_of(cell)], 1u); });
  __syncthreads();
  constexpr int S = kMaxChunks / kBoxDealThreads;  // counts -> first places, four per thread at a time
  static_assert(S == 4, "");
  unsigned all = 0;
  for (int i0 = 0; i0 < bins; i0 += kMaxChunks) {
    uint4* const mine_at = reinterpret_cast<uint4*>(place + i0 + t * S);
    const uint4 v = *mine_at;
    const unsigned mine = v.x + v.y + v.z + v.w;
    unsigned incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    if (i0) __syncthreads();
    if (lane == 63) wave_sum[wib] = incl;
    __syncthreads();
    unsigned at = all + incl - mine;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
      if (i < wib) at += wave_sum[i];
      all += wave_sum[i];
    }
    *mine_at = make_uint4(at, at + v.x, at + v.x + v.y, at + v.x + v.y + v.z);
  }
  __syncthreads();
  unsigned* const my_starts = starts + (long long)w * (bins + 1);
  for (int i = t; i < bins; i += kBoxDealThreads) my_starts[i] = place[i];
  if (t == 0) my_starts[bins] = all;
  __syncthreads();
  unsigned* const my_entries = entries + (long long)w * per;
  visit([&](unsigned cell) { my_entries[atomicAdd(&place[bin_of(cell)], 1u)] = cell; });
}

// One workgroup per chunk: its bits in LDS, from there with their prefixes to memory; base[group] = set bits of the group,
// totals[chunk] of all of them.  The windows of a chunk (of a sparse box) one after the other.  Where the box is too large, the coarse points go through the table instead (log_cap 0: it
// does not fit there).
__global__ void __launch_bounds__(kBitsThreads)
    k_box_bits(const Box* __restrict__ box_in, const unsigned* __restrict__ entries, const unsigned* __restrict__ starts, int dealers,
               int per, int log_chunks, Cells* __restrict__ cells, unsigned* __restrict__ base, unsigned* __restrict__ totals, const int4* __restrict__ coords, int n, int log_cap,
               unsigned long long* __restrict__ table, unsigned long long* __restrict__ ukeys, Ctl* ctl) {
  __shared__ __align__(16) unsigned bits[kLdsWords];
  constexpr int kWaves = kBitsThreads / 64, U = 4;
  __shared__ int before[kBoxDealers + 1], wave_sum[kWaves];
  __shared__ unsigned src[kBoxDealers], wave_bits[kWaves];
  const Box box = *box_in;
  const int t = threadIdx.x, lane = t & 63, wib = t >> 6;
  if (box.flags & (unsigned)FLAG_BOX) {
    if (log_cap) {
      const int each = (long long)gridDim.x * 256 >= n ? 256 : kBitsThreads;  // (few rows: to as many workgroups as there are)
      for (long long j0 = (long long)blockIdx.x * each; j0 < n; j0 += (long long)gridDim.x * each) {
        const long long j = t < each ? j0 + t : n;
        __syncthreads();
        coarse_unique<kWaves>(j < n, j < n ? coords[j] : make_int4(-1, 0, 0, 0), 2, table, log_cap, ukeys, ctl);
      }
    }
    return;
  }
  const unsigned groups = box.groups(), shift = box.shift, in_group = (1u << shift) - 1u;
  const unsigned n_groups = (groups + gridDim.x - 1) >> log_chunks;  // of this chunk (the last one may be beyond the box)
  if (blockIdx.x >= groups) {
    if (t == 0) totals[blockIdx.x] = 0;
    return;
  }
  unsigned total = 0;  // of this wave's groups
  const unsigned in_window = kLdsWords >> shift, windows = box.windows;
  for (unsigned g0 = 0, window = 0; g0 < n_groups; g0 += in_window, ++window) {
    int count = 0;
    if (t < dealers) {
      const unsigned* const s = starts + (long long)t * (gridDim.x * windows + 1) + blockIdx.x * windows + window;
      const unsigned a = s[0], b = s[1];
      src[t] = a;
      count = (int)(b - a);
    }
    int incl = count;
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    if (lane == 63) wave_sum[wib] = incl;
    const unsigned w0 = g0 << shift;
    const int here = (int)(min(in_window, n_groups - g0) << shift);
    for (int i = t; i < here / 4; i += kBitsThreads) reinterpret_cast<uint4*>(bits)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (t < kBoxDealers) {
      for (int i = 0; i < wib; ++i) incl += wave_sum[i];
      before[t + 1] = incl;
      if (t == 0) before[0] = 0;
    }
    __syncthreads();
    const int rows = before[kBoxDealers];
    auto set = [&](unsigned cell) {
      const unsigned word = cell >> 5, at = ((word >> shift >> log_chunks) << shift | (word & in_group)) - w0;
      if (at < (unsigned)here) atomicOr(&bits[at], 1u << (cell & 31));
    };
    // Many rows (a crowded window): a wave takes a dealer's at a time, which needs no search for the row's dealer.
    const bool crowded = rows > 64 * kBoxDealers;
    for (int w = wib; crowded && w < dealers; w += kWaves) {
      const int n_here = before[w + 1] - before[w];
      const unsigned* const mine = entries + (long long)w * per + src[w];
      for (int i0 = lane; i0 < n_here; i0 += U * 64) {
        unsigned cell[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cell[u] = i0 + u * 64 < n_here ? mine[i0 + u * 64] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i0 + u * 64 < n_here) set(cell[u]);
      }
    }
    for (int i0 = t; !crowded && i0 < rows; i0 += U * kBitsThreads) {
      int w[U] = {};  // the dealers: before[w] <= i < before[w + 1]
#pragma unroll
      for (int o = kBoxDealers / 2; o > 0; o >>= 1)
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (before[w[u] + o] <= i0 + u * kBitsThreads) w[u] += o;
      unsigned cell[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * kBitsThreads;
        cell[u] = i < rows ? entries[(long long)w[u] * per + src[w[u]] + (i - before[w[u]])] : 0u;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + u * kBitsThreads < rows) set(cell[u]);
    }
    __syncthreads();
    // a wave takes 256 consecutive words at a time, four to a lane: several groups, or a part of one, which it then takes whole
    const int unit = max(256, 1 << shift), seg = min(64, 1 << (shift - 2));
    for (int u0 = wib * unit; u0 < here; u0 += kWaves * unit) {
      unsigned run = 0;
      for (int i0 = u0; i0 < min(u0 + unit, here); i0 += 256) {
        const int i = i0 + 4 * lane;
        const uint4 v = i < here ? *reinterpret_cast<const uint4*>(bits + i) : make_uint4(0, 0, 0, 0);
        const unsigned n0 = __popc(v.x), n1 = n0 + __popc(v.y), n2 = n1 + __popc(v.z), n3 = n2 + __popc(v.w);
        unsigned in = n3;
        for (int o = 1; o < seg; o <<= 1) {
          const unsigned up = __shfl_up(in, o);
          if ((lane & (seg - 1)) >= o) in += up;
        }
        const unsigned b = run + in - n3, group = group_at(blockIdx.x, g0 + ((unsigned)i >> shift), log_chunks);
        const unsigned word = (group << shift) + ((unsigned)i & in_group);
        if (i < here && group < groups) {
          if (word < box.words) {  // (the buffer holds whole fours)
            uint4* const dst = reinterpret_cast<uint4*>(cells + word);
            dst[0] = make_uint4(v.x, b, v.y, b + n0);
            dst[1] = make_uint4(v.z, b + n1, v.w, b + n2);
          }
          if ((((unsigned)i + 4u) & in_group) == 0u) {
            base[group] = run + in;
            total += run + in;
          }
        }
        run += __shfl(in, 63);
      }
    }
    __syncthreads();
  }
  for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o);
  if (lane == 0) wave_bits[wib] = total;
  __syncthreads();
  if (t == 0) {
    for (int i = 1; i < kWaves; ++i) total += wave_bits[i];
    totals[blockIdx.x] = total;
  }
}

// base[group]: the set bits of the group become those before it (the first workgroup's work, four neighbouring groups to a lane, so that a
// line is read once: 200k rows 7.2 us, with up to 32 groups in a row per thread 8.0); the others preset the map (rows up to the padding).
__global__ void __launch_bounds__(kBaseThreads)
    k_box_base(const Box* __restrict__ box_in, const unsigned* __restrict__ totals, int chunks, unsigned* __restrict__ base, int V,
               uint4* __restrict__ map, unsigned* __restrict__ mask, Ctl* ctl) {
  constexpr int kWaves = kBaseThreads / 64, Q = kMaxGroups / kBaseThreads / 4, S = kMaxChunks / kBaseThreads;
  __shared__ unsigned sums[Q * kWaves], all;
  const int t = threadIdx.x, lane = t & 63, wib = t >> 6;
  const unsigned groups = box_in->groups();  // (no box: none, and no totals)
  auto scan = [&](unsigned incl) {
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    return incl;
  };
  if (blockIdx.x == 0) {
    uint4 v[Q];
    unsigned at[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const unsigned g = 4 * (q * kBaseThreads + t);
      v[q] = g < groups ? reinterpret_cast<const uint4*>(base)[g / 4] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const unsigned g = 4 * (q * kBaseThreads + t);  // (the last four may be incomplete)
      if (g + 1 >= groups) v[q].y = 0;
      if (g + 2 >= groups) v[q].z = 0;
      if (g + 3 >= groups) v[q].w = 0;
      const unsigned mine = v[q].x + v[q].y + v[q].z + v[q].w, incl = 4u * q * kBaseThreads < groups ? scan(mine) : 0u;
      if (lane == 63) sums[q * kWaves + wib] = incl;
      at[q] = incl - mine;
    }
    __syncthreads();
    if (wib == 0) {
      static_assert(Q * kWaves == 128, "two sums per lane");
      const unsigned a = sums[2 * lane], b = sums[2 * lane + 1], incl = scan(a + b);
      sums[2 * lane] = incl - a - b;
      sums[2 * lane + 1] = incl - b;
      if (lane == 63) all = incl;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const unsigned g = 4 * (q * kBaseThreads + t), x = at[q] + sums[q * kWaves + wib], y = x + v[q].x, z = y + v[q].y;
      if (g < groups) reinterpret_cast<uint4*>(base)[g / 4] = make_uint4(x, y, z, z + v[q].z);
    }
    const unsigned total = all;
    if (t == 0 && groups) ctl->count = total;  // (else: of the table's points, or none)
    if (total + t < (total + kRowPad - 1) / kRowPad * kRowPad) mask[total + t] = 0u;
    return;
  }
  unsigned mine = 0;
#pragma unroll
  for (int i = 0; i < S; ++i) mine += groups && i * kBaseThreads + t < chunks ? totals[i * kBaseThreads + t] : 0u;
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
  if (lane == 0) sums[wib] = mine;
  __syncthreads();
  unsigned total = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) total += sums[i];
  const unsigned rows_pad = (total + kRowPad - 1) / kRowPad * kRowPad;
  const long long vecs = (long long)rows_pad * V / 4, step = (long long)(gridDim.x - 1) * kBaseThreads;
  for (long long i = (long long)(blockIdx.x - 1) * kBaseThreads + t; i < vecs; i += step) map[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
}

// Row of a coarse point, or -1.
__device__ __forceinline__ int box_find(const Box& box, const Cells* cells, const unsigned* base, int b, int x, int y, int z) {
  if ((unsigned)(x - box.lo[1]) >= box.span[1] || (unsigned)(y - box.lo[2]) >= box.span[2] || (unsigned)(z - box.lo[3]) >= box.span[3]) return -1;
  const unsigned cell = cell_of(box, b, x, y, z);
  const Cells w = cells[cell >> 5];
  const unsigned before = base[cell >> (5 + box.shift)], bit = 1u << (cell & 31);
  return w.bits & bit ? (int)(before + w.before + (unsigned)__popc(w.bits & (bit - 1))) : -1;
}

// Outputs floor(p / 2) + (0 or 1 along each axis) that an input row of a stride-2 map may have an offset to.
constexpr int cands_of(int K) { return K == 3 ? 8 : 1; }

// The map from the input side (see k_scatter_down3), and the coarse points: every input meets the output floor(p / 2) (K = 2:
// only that one) and writes its coordinates; inputs of one output write the same (expanding the bits instead took 35 us where
// many stand in one word).
template <int K>
__global__ void __launch_bounds__(256)
    k_box_scatter(const int4* __restrict__ rows, int n_rows, const Box* __restrict__ box_in, const Cells* __restrict__ cells,
                  const unsigned* __restrict__ base, int* __restrict__ map, int4* __restrict__ coarse, int* __restrict__ cands, Ctl* ctl) {
  __shared__ unsigned wave_pairs[4];
  constexpr int LPR = cands_of(K), V = K * K * K;
  const Box box = *box_in;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long row = t / LPR;
  const int cand = K == 3 ? (int)(t & 7) : 0;
  bool found = false;
  int at = -1;
  if (row < n_rows && box.words) {
    const int4 c = rows[row];
    const int pc[3] = {c.y, c.z, c.w};
    int q[3], k = 0;
    bool ok = coord_ok(c.x, c.y, c.z, c.w);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int up = (cand >> (2 - a)) & 1;
      q[a] = (pc[a] >> 1) + up;
      const int d = pc[a] - 2 * q[a];
      ok = ok && d >= -1;  // (d <= 1 always)
      k = k * K + (K == 3 ? d + 1 : d);
    }
    if (ok) {
      const int n = box_find(box, cells, base, c.x, q[0], q[1], q[2]);
      if (n >= 0) {
        map[(long long)n * V + k] = (int)row;
        if (cand == 0) coarse[n] = make_int4(c.x, q[0], q[1], q[2]);
        found = true;
        at = n;
      }
    }
  }
  if (cands && row < n_rows) cands[t] = at;
  const unsigned long long bal = __ballot(found);
  if ((threadIdx.x & 63) == 0) wave_pairs[threadIdx.x >> 6] = (unsigned)__popcll(bal);
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned n = wave_pairs[0] + wave_pairs[1] + wave_pairs[2] + wave_pairs[3];
    if (n) atomicAdd(&ctl->pairs[(blockIdx.x % kPairSlots) * 16], (unsigned long long)n);
  }
}

// The parts of a stride-2 build's tables that are in use, into buffers of that size (16-byte words).
struct Copy3 {
  const uint4* src[3];
  uint4* dst[3];
  long long words[3];
};
__global__ void __launch_bounds__(256) k_copy3(const Copy3 c) {
  const long long step = (long long)gridDim.x * 256;
#pragma unroll
  for (int a = 0; a < 3; ++a)
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < c.words[a]; i += step) c.dst[a][i] = c.src[a][i];
}

// Plain fills (in place of memset calls, which must stay out of anything a caller may capture).
// The K = 1 map of a row set: row r meets itself; rows of the padding meet nothing.
__global__ void __launch_bounds__(256) k_identity_map(int* __restrict__ map, unsigned* __restrict__ mask,
                                                      long long rows, long long rows_pad) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows_pad) return;
  map[r] = r < rows ? (int)r : -1;
  mask[r] = r < rows ? 1u : 0u;
}

__global__ void __launch_bounds__(256) k_fill_u32(unsigned* __restrict__ dst, long long n, unsigned v) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = v;
}

// One launch that prepares a build: fills the table with ones (every key empty, every cell or value -1) and
// clears the control block.
// `marks` 16-byte words behind the table are cleared (k_filter_pack).
__global__ void __launch_bounds__(256) k_build_init(ulonglong2* __restrict__ tab, long long words, int marks, Ctl* ctl) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long long i = t; i < words; i += stride) tab[i] = make_ulonglong2(kEmpty, kEmpty);
  for (long long i = t; i < marks; i += stride) tab[words + i] = make_ulonglong2(0ull, 0ull);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      ctl->flags = 0;
      ctl->count = 0;
      ctl->tick_top = 0;
    }
    if (threadIdx.x < kPairSlots) {
      ctl->pairs[threadIdx.x * 16] = 0;
      ctl->entries[threadIdx.x * 16] = 0;
      ctl->key_or[threadIdx.x * 16] = 0;
      ctl->key_and[threadIdx.x * 16] = ~0ull;
    }
  }
}

// The figures of a build straight into pinned host memory, where the host polls for them: a copy and a stream synchronisation in
// their place cost about 20 us of idle GPU per use.  One wave; all its loads are in flight together, and where the figures fit into words of
// eight bytes, each with a ready bit of its own, nothing waits for a store to arrive (a fence between figures and a flag took 1.5 us).
enum Publish {
  kPublishWord,     // flags and pairs
  kPublishOutputs,  // and the number of outputs; rows that share an entry are flagged
  kPublishAll,      // everything, behind a fence
  kPublishEnd       // nothing: the kernels before this one have ended (a submanifold probe stores the word itself)
};
template <Publish WHAT> __global__ void __launch_bounds__(64) k_publish(const Ctl* __restrict__ ctl, HostResult* host) {
  const int lane = threadIdx.x;  // kPairSlots == 64
  if constexpr (WHAT == kPublishEnd) {
    if (lane == 0) __hip_atomic_store(&host->ready, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return;
  }
  const unsigned long long mine = ctl->pairs[lane * 16] & ((1ull << 40) - 1);  // (above: publish_pairs' arrivals)
  unsigned long long pairs = mine, flags = ctl->flags, count = 0, entries = 0, k_or = 0, k_and = ~0ull;
  if constexpr (WHAT != kPublishWord) count = ctl->count, entries = ctl->entries[lane * 16];
  if constexpr (WHAT == kPublishAll) k_or = ctl->key_or[lane * 16], k_and = ctl->key_and[lane * 16];
  for (int o = 32; o > 0; o >>= 1) {
    pairs += __shfl_xor(pairs, o);
    if constexpr (WHAT != kPublishWord) entries += __shfl_xor(entries, o);
    if constexpr (WHAT == kPublishAll) {
      k_or |= __shfl_xor(k_or, o);
      k_and &= __shfl_xor(k_and, o);
    }
  }
  if constexpr (WHAT != kPublishAll) {
    if (WHAT == kPublishOutputs && entries != pairs) flags |= FLAG_DUP;
    if (lane == 0) {
      if (WHAT == kPublishOutputs) __hip_atomic_store(&host->outputs, kHostReady | count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(&host->word, kHostReady | ((flags & 0xFFu) << 48) | (pairs & 0xFFFFFFFFFFFFull), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  for (int g = 0; g < 5; ++g) {
    unsigned long long v = lane / kPlaneSlots == g ? mine : 0ull;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) host->plane_pairs[g] = v;
  }
  if (lane == 0) {
    host->flags = flags;
    host->count = count;
    host->key_or = k_or;
    host->key_and = k_and;
    host->pairs = pairs;
    host->entries = entries;
    __threadfence_system();
    __hip_atomic_store(&host->ready, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ---- submanifold 5x5x5 build over a table of z-runs ----
// One table entry holds four cells that are neighbours along z: the key is (b, x, y, z >> 2) and
// rows[z & 3] the input row there.  A voxel's five neighbours in a column (x + dx, y + dy,
// z - 2 .. z + 2) lie in two entries, so the whole neighbourhood takes 50 entry reads.  Each row then
// writes its own map entries and masks: no entry of another row is touched, so the maps need no preset and the
// masks no atomics.
struct RunSlot {
  unsigned long long key;
  int rows[4];
  unsigned long long pad;
};
static_assert(sizeof(RunSlot) == 32, "two entries per 64-byte line");

// (32-bit mixing: a 64-bit multiply costs several times as many instructions, and the probe hashes
// twice per lane)
__device__ __forceinline__ unsigned hash_run(unsigned long long key) {
  unsigned h = (unsigned)key * 0x9E3779B1u ^ (unsigned)(key >> 32) * 0x85EBCA77u;
  h ^= h >> 15;
  return h * 0xC2B2AE3Du;
}
__device__ __forceinline__ unsigned hash_slot(unsigned long long key, int log_cap) { return hash_run(key) >> (32 - log_cap); }

// Which runs exist, one bit per hash value: 128 KB, which a workgroup of the probe holds in LDS.  Of the 50 entries that a
// row looks up most do not exist, and the filter lets only 7 to 15 % of the absent ones through.  The insert marks bytes (plain
// stores: every writer stores the same, and an atomic per row costs 1 us for 10,000), k_filter_pack makes bits of them.
constexpr int kFilterBits = 20;
constexpr int kMarkWords = (1 << kFilterBits) / 16, kFilterWords = (1 << kFilterBits) / 32;
__device__ __forceinline__ unsigned filter_bit(unsigned hash) { return hash >> (32 - kFilterBits); }

__global__ void __launch_bounds__(256) k_filter_pack(const uint4* __restrict__ marks, unsigned* __restrict__ bits) {
  const int i = blockIdx.x * 256 + threadIdx.x;  // (kFilterWords threads)
  const uint4 a = marks[2 * i], b = marks[2 * i + 1];
  const unsigned v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  unsigned w = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) w |= ((v[u] & 1u) | ((v[u] >> 7) & 2u) | ((v[u] >> 14) & 4u) | ((v[u] >> 21) & 8u)) << (4 * u);
  bits[i] = w;
}

// The table arrives filled with ones: every key empty, every cell -1.  Duplicate rows store into
// one cell; the probe notices, because one of them no longer finds itself there.
__global__ void __launch_bounds__(256) k_insert_runs(const int4* __restrict__ coords, int n, RunSlot* tab, int log_cap,
                                                     Ctl* ctl, int4* __restrict__ keep, unsigned char* marks) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int4 c = coords[j];
  keep[j] = c;  // the kmap's own copy of the caller's rows
  if (!coord_ok(c.x, c.y, c.z, c.w)) {
    atomicOr(&ctl->flags, FLAG_RANGE);
    return;
  }
  const unsigned long long key = pack_key(c.x, c.y, c.z, c.w >> 2);
  const unsigned slot_mask = (1u << log_cap) - 1u, h = hash_run(key);
  if (marks) marks[filter_bit(h)] = 1;
  unsigned s = h >> (32 - log_cap);
  for (unsigned it = 0; it <= slot_mask; ++it) {
    const unsigned long long old = atomicCAS(&tab[s].key, kEmpty, key);
    if (old == kEmpty || old == key) {
      tab[s].rows[c.w & 3] = j;
      return;
    }
    s = (s + 1) & slot_mask;
  }
  atomicOr(&ctl->flags, FLAG_FULL);
}

// Finishes a lookup whose first entry (slot s) is already loaded: a = key and cells 0, 1.
__device__ __forceinline__ void run_resolve(const RunSlot* tab, int log_cap, unsigned long long key, unsigned s,
                                            uint4 a, int cells[4]) {
  const unsigned slot_mask = (1u << log_cap) - 1u;
  for (unsigned it = 0; it <= slot_mask; ++it) {
    const unsigned long long k = (unsigned long long)a.x | ((unsigned long long)a.y << 32);
    if (k == key) {
      const uint2 b = *reinterpret_cast<const uint2*>(&tab[s].rows[2]);
      cells[0] = (int)a.z;
      cells[1] = (int)a.w;
      cells[2] = (int)b.x;
      cells[3] = (int)b.y;
      return;
    }
    if (k == kEmpty) return;
    s = (s + 1) & slot_mask;
    a = *reinterpret_cast<const uint4*>(tab + s);
  }
}

// The neighbours of a row in column (tx, ty): cells z - 2 .. z + 2.  They are five in a row of the window [run q_lo | run
// q_lo + 1], starting at (z - 2) & 3.  (z itself is in range, so the runs' indices fit the key's field; cells beside the
// range are dropped.)  FILTER: absent runs are mostly known without a look at the table.
template <bool FILTER>
__device__ __forceinline__ void probe_column(int b, int tx, int ty, int z, const RunSlot* __restrict__ tab, int log_cap,
                                             const unsigned* filter, int* nb) {
  const int q_lo = (z - 2) >> 2, i0 = (z - 2) & 3;
  const unsigned long long key_lo = pack_key(b, tx, ty, q_lo), key_hi = key_lo + 1;
  const unsigned h_lo = hash_run(key_lo), h_hi = hash_run(key_hi);
  const unsigned s_lo = h_lo >> (32 - log_cap), s_hi = h_hi >> (32 - log_cap);
  int w[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
  if constexpr (!FILTER) {
    // (cells 2 and 3 are fetched only where the key matches: without the filter most entries are not there)
    const uint4 a_lo = *reinterpret_cast<const uint4*>(tab + s_lo);  // both in flight
    const uint4 a_hi = *reinterpret_cast<const uint4*>(tab + s_hi);
    run_resolve(tab, log_cap, key_lo, s_lo, a_lo, w);
    run_resolve(tab, log_cap, key_hi, s_hi, a_hi, w + 4);
  } else {
    const unsigned f_lo = filter_bit(h_lo), f_hi = filter_bit(h_hi);
    bool want_lo = (filter[f_lo >> 5] >> (f_lo & 31)) & 1u, want_hi = (filter[f_hi >> 5] >> (f_hi & 31)) & 1u;
    const unsigned slot_mask = (1u << log_cap) - 1u;
    unsigned at_lo = s_lo, at_hi = s_hi;
    // both runs advance together: a wave's lookups take as many rounds as the longest chain of any of them
    for (unsigned it = 0; it <= slot_mask && (want_lo || want_hi); ++it) {
      uint4 a_lo, a_hi;
      uint2 b_lo, b_hi;
      if (want_lo) {
        a_lo = *reinterpret_cast<const uint4*>(tab + at_lo);
        b_lo = *reinterpret_cast<const uint2*>(&tab[at_lo].rows[2]);
      }
      if (want_hi) {
        a_hi = *reinterpret_cast<const uint4*>(tab + at_hi);
        b_hi = *reinterpret_cast<const uint2*>(&tab[at_hi].rows[2]);
      }
      if (want_lo) {
        const unsigned long long k = (unsigned long long)a_lo.x | ((unsigned long long)a_lo.y << 32);
        if (k == key_lo) w[0] = (int)a_lo.z, w[1] = (int)a_lo.w, w[2] = (int)b_lo.x, w[3] = (int)b_lo.y;
        want_lo = k != key_lo && k != kEmpty;
        at_lo = (at_lo + 1) & slot_mask;
      }
      if (want_hi) {
        const unsigned long long k = (unsigned long long)a_hi.x | ((unsigned long long)a_hi.y << 32);
        if (k == key_hi) w[4] = (int)a_hi.z, w[5] = (int)a_hi.w, w[6] = (int)b_hi.x, w[7] = (int)b_hi.y;
        want_hi = k != key_hi && k != kEmpty;
        at_hi = (at_hi + 1) & slot_mask;
      }
    }
  }
  const bool b1 = i0 & 1, b2 = i0 & 2;
#pragma unroll
  for (int d = 0; d < 5; ++d) {
    const int v = b2 ? (b1 ? w[3 + d] : w[2 + d]) : (b1 ? w[1 + d] : w[d]);
    nb[d] = coord_ok(b, tx, ty, z + d - 2) ? v : -1;
  }
}

constexpr int kProbeThreads = 1024;  // with the filter: one workgroup per CU
// The filter into LDS.
__device__ __forceinline__ void load_filter(const unsigned* __restrict__ bits, unsigned* lds) {
  constexpr int U = kFilterWords / 4 / kProbeThreads;
  uint4 v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = reinterpret_cast<const uint4*>(bits)[u * kProbeThreads + threadIdx.x];
#pragma unroll
  for (int u = 0; u < U; ++u) reinterpret_cast<uint4*>(lds)[u * kProbeThreads + threadIdx.x] = v[u];
  __syncthreads();
}

// ---- submanifold 3x3x3 builds in buckets ----
// The rows are dealt into buckets by the block of 8 x 8 x 8 cells that they lie in (hashed: several blocks share a bucket), and a
// row at a face of its block is copied into the neighbours' buckets as well.  A row's whole neighbourhood then lies in its own
// bucket, and one workgroup per bucket hashes the bucket into LDS and looks its rows up there: no table in memory that has to be
// cleared, no atomic and no look-up that leaves the CU.  The table in LDS holds runs of four cells along z: a voxel's three neighbours
// in a column (x + dx, y + dy, z - 1 .. z + 1) lie in one run, or in two when the range crosses a multiple of four.  Each row writes its
// own 27 map entries and its own mask: no entry of another row is touched, so the map needs no preset and the masks no atomics.
// GPU time of unwaited builds, a table of runs in memory (cleared, filled with an atomic per row, probed with 13.5 reads per row
// of which a filter in LDS answered some) and so, us: a scan of 30k rows 28, 17; 60k 36, 25; 100k 44, 28.5; 200k 67, 45; 400k
// 115, 71; a room of 60k 32, 27; 100k 41.5, 37; 300k 83, 63; 7k rows 18, 14.  What bounds it: round trips behind barriers (the waves of
// k_probe_buckets wait in 6 of 10 cycles, with 14 reads in flight per CU, 1.6 TB/s and 1 % of the cycles waiting for LDS; a block holds
// up to 100 rows of a surface, and buckets of 256 rows on average up to 700), and launch and publication, 5 us.  Behind the table only on
// full grids, whose blocks have 512 rows and as many copies, so that few workgroups have all the work: waited builds of cubes of 27k rows 41,
// 49; 300k 112, 149; 2.1M 711, 556; a full plane of 400k 111, 92.
constexpr int kBlockBits = 3;      // (16 cells a side: 1.5 copies of a row in place of 2, but buckets of up to 1,800 rows: 300k rows of a room 124 us)
constexpr int kDealThreads = 512;
constexpr int kDealers = 256;      // workgroups of k_deal_rows at most
constexpr int kCopies = 8;         // buckets that a row may be dealt into
constexpr int kMaxBucketBits = 14;
// (1,024 threads: 100k rows 31 us; 512: three workgroups fit on a CU and take longer than two of 768 by more than that)
constexpr int kBucketThreads = 768;
constexpr int kOwnRows = 512;      // rows of a bucket whose coordinates are in LDS at a time
constexpr int kBucketRows = 1536;  // rows of a bucket, with the copies, that are in the table at a time
constexpr int kRunSlotBits = 11;
static_assert(kBucketRows < (1 << kRunSlotBits), "every chain of slots ends");
__host__ __device__ constexpr int deal_lds(int log_b) { return (2 << log_b) * 4; }

struct Dealt {
  unsigned lo, hi;  // the key
  int row;
};

__device__ __forceinline__ unsigned bucket_of(int b, int x, int y, int z, int log_b) {
  return hash_run(pack_key(b, x, y, z)) >> (32 - log_b);
}

// f(bucket, halo) for every bucket that a row is dealt into, once each; the row's own one first.
template <typename F> __device__ __forceinline__ void for_buckets(int4 c, int log_b, F f) {
  constexpr int S = 1 << kBlockBits;
  const int p[3] = {c.y, c.z, c.w};
  int q[3], d[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int o = p[a] & (S - 1);
    q[a] = p[a] >> kBlockBits;
    d[a] = o == 0 ? -1 : o == S - 1 ? 1 : 0;
  }
  unsigned seen[kCopies];
  seen[0] = bucket_of(c.x, q[0], q[1], q[2], log_b);
  f(seen[0], 0);
#pragma unroll
  for (int m = 1; m < kCopies; ++m) {
    seen[m] = seen[0];
    if (((m & 1) && !d[0]) || ((m & 2) && !d[1]) || ((m & 4) && !d[2])) continue;
    const unsigned to = bucket_of(c.x, q[0] + (m & 1 ? d[0] : 0), q[1] + (m & 2 ? d[1] : 0), q[2] + (m & 4 ? d[2] : 0), log_b);
    bool fresh = true;
#pragma unroll
    for (int i = 0; i < m; ++i) fresh = fresh && to != seen[i];
    if (!fresh) continue;
    seen[m] = to;
    f(to, 1);
  }
}

// Workgroup w deals rows [w per, w per + per) and leaves those of buckets [part 2^log_b, part 2^log_b + 2^log_b), ordered by bucket (a
// bucket's own rows before the copies), at entries + 8 per w; starts[w][2 bucket + copies] says where each begins.  The first part also
// makes the kmap's own copy of the caller's rows, the map of the padding and of rows beside the range (no neighbours; they fail the
// build), and clears the control block.
template <bool PARTS>
__global__ void __launch_bounds__(kDealThreads)
    k_deal_rows(const int4* __restrict__ coords, int n, int per, int log_b, int log_parts, unsigned part_of, Dealt* __restrict__ entries, unsigned* __restrict__ starts,
                unsigned* __restrict__ dealer_flags, int4* __restrict__ keep, long long rows_pad, int* __restrict__ map,
                unsigned* __restrict__ mask, Ctl* ctl) {
  constexpr int V = 27, U = 2;
  const unsigned part = PARTS ? part_of : 0u;
  extern __shared__ __align__(16) unsigned place[];  // [2 << log_b]
  __shared__ unsigned wave_sum[kDealThreads / 64], flags;
  const int t = threadIdx.x, lane = t & 63, wib = t >> 6, w = blockIdx.x;
  const int cells = 2 << log_b;
  const int first = (int)min((long long)w * per, (long long)n), last = (int)min((long long)first + per, (long long)n);
  for (int i = t; i < cells; i += kDealThreads) place[i] = 0;
  if (t == 0) flags = 0;
  __syncthreads();
  auto visit = [&](auto f) {
    for (long long r0 = first + t; r0 < last; r0 += U * kDealThreads) {
      int4 c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) c[u] = r0 + u * kDealThreads < last ? coords[r0 + u * kDealThreads] : make_int4(-1, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (r0 + u * kDealThreads < last) f((int)r0 + u * kDealThreads, c[u]);
    }
  };
  auto visit_copies = [&](int4 c, auto f) {  // f(place)
    for_buckets(c, PARTS ? log_b + log_parts : log_b, [&](unsigned b, int halo) {
      if constexpr (PARTS) {
        if (b >> log_b != part) return;
        b &= (1u << log_b) - 1u;
      }
      f(2 * b + halo);
    });
  };
  visit([&](int r, int4 c) {
    if (part == 0) keep[r] = c;
    if (coord_ok(c.x, c.y, c.z, c.w)) {
      visit_copies(c, [&](unsigned at) { atomicAdd(&place[at], 1u); });
    } else if (part == 0) {
      flags = (unsigned)FLAG_RANGE;
      for (int k = 0; k < V; ++k) map[(long long)r * V + k] = -1;
      mask[r] = 0u;
    }
  });
  __syncthreads();
  if (t == 0 && part == 0) dealer_flags[w] = flags;
  // counts -> first places, as many cells per thread as there are, four at a time
  const int share = max(cells / kDealThreads, 4), c0 = min(t * share, cells), c1 = min(c0 + share, cells);
  unsigned mine = 0;
  for (int i = c0; i < c1; i += 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(place + i);
    mine += v.x + v.y + v.z + v.w;
  }
  unsigned incl = mine;
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wave_sum[wib] = incl;
  __syncthreads();
  unsigned at = incl - mine, all = 0;
  for (int i = 0; i < kDealThreads / 64; ++i) {
    if (i < wib) at += wave_sum[i];
    all += wave_sum[i];
  }
  for (int i = c0; i < c1; i += 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(place + i);
    *reinterpret_cast<uint4*>(place + i) = make_uint4(at, at + v.x, at + v.x + v.y, at + v.x + v.y + v.z);
    at += v.x + v.y + v.z + v.w;
  }
  __syncthreads();
  unsigned* const my_starts = starts + (long long)w * (cells + 1);
  for (int i = t; i < cells; i += kDealThreads) my_starts[i] = place[i];
  if (t == 0) my_starts[cells] = all;
  __syncthreads();
  Dealt* const my_entries = entries + (long long)w * per * kCopies;
  visit([&](int r, int4 c) {
    if (!coord_ok(c.x, c.y, c.z, c.w)) return;
    const unsigned long long key = pack_key(c.x, c.y, c.z, c.w);
    const Dealt e{(unsigned)key, (unsigned)(key >> 32), r};
    visit_copies(c, [&](unsigned at) { my_entries[atomicAdd(&place[at], 1u)] = e; });
  });
  if (part) return;
  if (w == 0) {
    if (t == 0) ctl->flags = 0, ctl->count = 0, ctl->tick_top = 0;
    if (t < kPairSlots) {
      ctl->pairs[t * 16] = 0;
      ctl->entries[t * 16] = 0;
      ctl->key_or[t * 16] = 0;
      ctl->key_and[t * 16] = ~0ull;
    }
  }
  if (w == (int)gridDim.x - 1) {
    for (long long i = (long long)n * V + t; i < rows_pad * V; i += kDealThreads) map[i] = -1;
    if (n + t < rows_pad) mask[n + t] = 0u;  // (fewer than kRowPad)
  }
}

// The workgroup that arrives last sums the pair counters and writes the result into pinned host
// memory.  A pair slot is one 64-bit counter: pairs in its low 40 bits, arrivals above, so that one
// atomic both adds the workgroup's pairs and tells it whether it was the slot's last (a second
// level counts the finished slots: no address sees more than gridDim/64 or 64 atomics).  Called by
// the first wave only, after the others have left: two returning atomics in a row, awaited by the
// whole workgroup, would keep all of its waves.  Every value the last workgroup
// reads was produced by an atomic whose return its producer waited for before counting itself in,
// and is read with an atomic, so no cache write-back is needed.  launches: one after the other, of equal grids.
__device__ __forceinline__ void publish_pairs(unsigned wg_pairs, unsigned wg_flags, unsigned launches, Ctl* ctl, HostResult* host) {
  constexpr unsigned long long kArrive = 1ull << 40;
  int last = 0;
  if (threadIdx.x == 0) {
    unsigned long long before = wg_flags ? atomicOr(&ctl->flags, (unsigned long long)wg_flags) : 0ull;
    asm volatile("" : "+v"(before));  // (the flags have arrived)
    const unsigned slot = blockIdx.x % kPairSlots;
    before = atomicAdd(&ctl->pairs[slot * 16], (unsigned long long)wg_pairs + kArrive);
    const unsigned slot_wgs = (gridDim.x - slot + kPairSlots - 1) / kPairSlots;
    const unsigned used_slots = gridDim.x < (unsigned)kPairSlots ? gridDim.x : (unsigned)kPairSlots;
    if ((unsigned)(before >> 40) + 1 == slot_wgs * launches) last = atomicAdd(&ctl->tick_top, 1u) + 1 == used_slots;
  }
  last = __builtin_amdgcn_readfirstlane(last);
  if (last) {
    unsigned long long v = atomicAdd(&ctl->pairs[threadIdx.x * 16], 0ull) & (kArrive - 1);  // kPairSlots == 64 lanes
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (threadIdx.x == 0)
      host->word = kHostReady | ((atomicOr(&ctl->flags, 0ull) & 0xFFull) << 48) | (v & 0xFFFFFFFFFFFFull);
  }
}

__device__ __forceinline__ unsigned spread3(unsigned g) {  // bit c of 9 -> bit 3c
  g = (g | (g << 16)) & 0x030000FFu;
  g = (g | (g << 8)) & 0x0300F00Fu;
  g = (g | (g << 4)) & 0x030C30C3u;
  return (g | (g << 2)) & 0x09249249u;
}

// A run of the table in LDS: the key, and the places in the bucket of the rows in its four cells (16 bits each).
struct __align__(16) BucketRun {
  unsigned long long key, cells;
};
constexpr unsigned kNoCell = 0xFFFFu;

// The places of a row's neighbours in column (tx, ty): cells z - 1 .. z + 1, three in a row of the window [run q_lo | run q_lo + 1],
// starting at (z - 1) & 3.  (z itself is in range, so the runs' indices fit the key's field; cells beside the range are dropped.)
__device__ __forceinline__ void probe_bucket_column(int b, int tx, int ty, int z, const BucketRun* tab, unsigned* cell) {
  constexpr unsigned slot_mask = (1u << kRunSlotBits) - 1u;
  const int q_lo = (z - 1) >> 2, i0 = (z - 1) & 3;
  const unsigned long long key = pack_key(b, tx, ty, q_lo);
  unsigned s_lo = hash_run(key) >> (32 - kRunSlotBits), s_hi = hash_run(key + 1) >> (32 - kRunSlotBits);
  unsigned long long lo = ~0ull, hi = ~0ull;
  bool want_lo = true, want_hi = i0 + 3 > 4;
  for (unsigned it = 0; it <= slot_mask && (want_lo || want_hi); ++it) {  // both advance together
    const BucketRun e_lo = tab[s_lo], e_hi = tab[s_hi];
    if (want_lo && e_lo.key == key) lo = e_lo.cells;
    if (want_hi && e_hi.key == key + 1) hi = e_hi.cells;
    want_lo = want_lo && e_lo.key != key && e_lo.key != kEmpty;
    want_hi = want_hi && e_hi.key != key + 1 && e_hi.key != kEmpty;
    s_lo = (s_lo + 1) & slot_mask;
    s_hi = (s_hi + 1) & slot_mask;
  }
  const int sh = i0 * 16;
  const unsigned long long w = sh ? (lo >> sh) | (hi << (64 - sh)) : lo;
#pragma unroll
  for (int d = 0; d < 3; ++d) cell[d] = coord_ok(b, tx, ty, z + d - 1) ? (unsigned)(w >> (16 * d)) & 0xFFFFu : kNoCell;
}

// One workgroup per bucket; nine lanes per row, one per column (dx, dy), seven rows per wave.  kBucketRows rows of the bucket are in the
// table at a time, kOwnRows of those that are looked up in LDS: a bucket is almost always within both, and one of any size is walked
// in as many rounds as it takes.  Rows that stand in one cell all lie in one bucket (rows padded with zeros: any number of them, and the
// rounds grow with its square), so a bucket of several rounds is left as soon as one has shown two such rows: the build fails, and the
// rows that were not looked up have no neighbours.
__global__ void __launch_bounds__(kBucketThreads)
    k_probe_buckets(const Dealt* __restrict__ entries, const unsigned* __restrict__ starts, const unsigned* __restrict__ dealer_flags,
                    int dealers, int per, int log_b, unsigned parts, int* __restrict__ map, unsigned* __restrict__ mask, Ctl* ctl,
                    HostResult* host) {
  constexpr int V = 27, LPR = 9, RPW = 7, kWaves = kBucketThreads / 64;
  constexpr unsigned slot_mask = (1u << kRunSlotBits) - 1u;
  __shared__ BucketRun tab[1 << kRunSlotBits];
  __shared__ Dealt own[kOwnRows];
  __shared__ int row_of[kBucketRows];
  // rows of a bucket: its own ones dealer by dealer, then the copies; [.][w]: how many before dealer w's, and where they stand
  __shared__ int before[2][kDealers + 1];
  __shared__ unsigned src[2][kDealers];
  __shared__ int wave_sum[2][kDealers / 64];
  __shared__ unsigned wave_pairs[kWaves], s_flags;
  static_assert(kBucketThreads >= kDealers, "a thread per dealer");
  const int t = threadIdx.x, lane = t & 63, wib = t >> 6;
  const int cells = 2 << log_b;
  if (t == 0) s_flags = 0;
  int n[2] = {0, 0}, incl[2];
  if (t < dealers) {
    const unsigned* const s = starts + (long long)t * (cells + 1) + 2 * blockIdx.x;
    const unsigned a = s[0], b = s[1], c = s[2];
    src[0][t] = a, src[1][t] = b;
    n[0] = (int)(b - a), n[1] = (int)(c - b);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    incl[h] = n[h];
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl[h], o);
      if (lane >= o) incl[h] += up;
    }
    if (t < kDealers && lane == 63) wave_sum[h][wib] = incl[h];
  }
  __syncthreads();
  if (t < kDealers) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int at = incl[h];
      for (int i = 0; i < wib; ++i) at += wave_sum[h][i];
      before[h][t + 1] = at;
      if (t == 0) before[h][0] = 0;
    }
  }
  __syncthreads();
  const int n_own = before[0][kDealers], n_all = n_own + before[1][kDealers];
  const bool rounds = __builtin_expect(n_all > kBucketRows, 0);
  auto entry = [&](int i) {
    const int h = i >= n_own ? 1 : 0;
    const int j = h ? i - n_own : i;
    int w = 0;  // the dealer: before[h][w] <= j < before[h][w + 1]
#pragma unroll
    for (int o = kDealers / 2; o > 0; o >>= 1)
      if (before[h][w + o] <= j) w += o;
    return entries[(long long)w * per * kCopies + src[h][w] + (j - before[h][w])];
  };
  const int sub = lane / LPR, col = lane - sub * LPR;
  auto run_of = [](const Dealt& e) {
    const unsigned long long key = (unsigned long long)e.lo | ((unsigned long long)e.hi << 32);
    return (key & ~0xFFFFull) | (unsigned)((((int)(e.lo & 0xFFFFu) - 32768) >> 2) + 32768);
  };
  unsigned pairs = 0, bad = 0;
  int looked_up = 0;  // own rows that have their map rows
  bool leave = false;
  for (int c0 = 0; n_own && !leave && (c0 == 0 || c0 < n_all); c0 += kBucketRows) {
    const int in_table = min(kBucketRows, n_all - c0);
    if (c0) __syncthreads();
    for (int i = t; i <= (int)slot_mask; i += kBucketThreads) reinterpret_cast<ulonglong2*>(tab)[i] = make_ulonglong2(kEmpty, ~0ull);
    __syncthreads();
    for (int i = t; i < in_table; i += kBucketThreads) {
      const Dealt e = entry(c0 + i);
      row_of[i] = e.row;
      if (c0 == 0 && i < kOwnRows && i < n_own) own[i] = e;
      const unsigned long long run = run_of(e);
      unsigned s = hash_run(run) >> (32 - kRunSlotBits);
      for (unsigned it = 0; it <= slot_mask; ++it) {
        const unsigned long long old = atomicCAS(&tab[s].key, kEmpty, run);
        if (old == kEmpty || old == run) {
          reinterpret_cast<unsigned short*>(&tab[s].cells)[e.lo & 3u] = (unsigned short)i;
          break;
        }
        s = (s + 1) & slot_mask;
      }
    }
    if (rounds) {  // a row (or a copy) whose place another one has taken
      __syncthreads();
      for (int i = t; i < in_table; i += kBucketThreads) {
        const Dealt e = entry(c0 + i);
        const unsigned long long run = run_of(e);
        unsigned s = hash_run(run) >> (32 - kRunSlotBits);
        for (unsigned it = 0; it <= slot_mask && tab[s].key != run; ++it) s = (s + 1) & slot_mask;
        if (((unsigned)(tab[s].cells >> (16 * (e.lo & 3u))) & 0xFFFFu) != (unsigned)i) bad = (unsigned)FLAG_DUP;
      }
      if (bad) atomicOr(&s_flags, bad);
    }
    for (int o0 = 0; o0 < n_own; o0 += kOwnRows) {
      const int n_here = min(kOwnRows, n_own - o0);
      if (rounds || o0) {
        __syncthreads();
        leave = rounds && s_flags;  // (nobody writes it between this barrier and the next)
        if (leave) break;
        for (int i = t; i < n_here; i += kBucketThreads) own[i] = entry(o0 + i);
      }
      __syncthreads();
      for (int i0 = wib * RPW; i0 < n_here; i0 += kWaves * RPW) {
        const int i = i0 + sub;
        const bool active = sub < RPW && i < n_here;
        const Dealt e = own[active ? i : 0];
        const int row = e.row, b = (int)(e.hi >> 16), x = (int)(e.hi & 0xFFFFu) - 32768, y = (int)(e.lo >> 16) - 32768,
                  z = (int)(e.lo & 0xFFFFu) - 32768;
        const int tx = x + col / 3 - 1, ty = y + col % 3 - 1;
        unsigned cell[3] = {kNoCell, kNoCell, kNoCell};
        if (active && coord_ok(b, tx, ty, z)) probe_bucket_column(b, tx, ty, z, tab, cell);
        // a row that does not find itself at its own place shares it with another row
        if (active && col == 4) {
          const int mine = o0 + i - c0;
          if (cell[1] != (mine >= 0 && mine < in_table ? (unsigned)mine : kNoCell)) bad = (unsigned)FLAG_DUP;
        }
        int nb[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) nb[d] = cell[d] == kNoCell ? -1 : row_of[cell[d]];
        if (active) {
          int* const dst = map + (long long)row * V + 3 * col;
#pragma unroll
          for (int d = 0; d < 3; ++d)
            if (c0 == 0 || nb[d] >= 0) dst[d] = nb[d];
        }
        const unsigned long long b0 = __ballot(nb[0] >= 0), b1 = __ballot(nb[1] >= 0), b2 = __ballot(nb[2] >= 0);
        pairs += (unsigned)(__popcll(b0) + __popcll(b1) + __popcll(b2));
        if (active && col == 0) {
          const int sh = sub * LPR;
          const unsigned m = spread3((unsigned)(b0 >> sh) & 0x1FFu) | (spread3((unsigned)(b1 >> sh) & 0x1FFu) << 1) |
                             (spread3((unsigned)(b2 >> sh) & 0x1FFu) << 2);
          mask[row] = c0 ? mask[row] | m : m;
        }
      }
      if (c0 == 0) looked_up = o0 + n_here;
      if (rounds && bad) atomicOr(&s_flags, bad);
    }
  }
  if (leave)
    for (int i = looked_up + t; i < n_own; i += kBucketThreads) {
      const int row = entry(i).row;
      for (int k = 0; k < V; ++k) map[(long long)row * V + k] = -1;
      mask[row] = 0u;
    }
  if (blockIdx.x == 0 && t < dealers) bad |= dealer_flags[t];
  if (lane == 0) wave_pairs[wib] = pairs;
  if (bad) atomicOr(&s_flags, bad);
  __syncthreads();
  if (t >= 64) return;
  unsigned sum = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) sum += wave_pairs[w];
  publish_pairs(sum, s_flags, parts, ctl, host);
}

// ---- small submanifold 3x3x3 builds in one launch ----
// Up to kSmallRows rows every workgroup hashes all of them into a table of its own in LDS and looks its share of the rows up
// there: nothing is cleared beforehand, no atomic leaves the CU, and no launch waits for another.  A slot holds the row and 19
// bits of its hash, so that a lookup compares keys only where it has most likely found its row.  Whole builds, us: 500 rows 37
// -> 21, 2k 36 -> 23, 5k 32 -> 27; at 7k 34 and 32, at 9k 32 and 43: every workgroup inserts all rows, one after the other per
// thread.
constexpr int kSmallRows = 5120, kSmallThreads = 1024, kSmallWgs = kPairSlots;
constexpr int kSmallRowBits = 13;
constexpr unsigned kSmallEmpty = ~0u;
static_assert(kSmallRows < (1 << kSmallRowBits) - 1, "a slot is never mistaken for an empty one");
__host__ __device__ constexpr int small_slots(int n) {
  int c = 1024;
  while (c < 2 * n) c *= 2;
  return c;
}
__global__ void __launch_bounds__(kSmallThreads)
    k_build_small3(const int4* __restrict__ rows, int n, int rows_pad, int4* __restrict__ keep, int* __restrict__ map,
                   unsigned* __restrict__ mask, Ctl* ctl) {
  constexpr int V = 27, RPW = 2, kWaves = kSmallThreads / 64;
  extern __shared__ __align__(16) unsigned long long keys[];  // [n], then the slots
  __shared__ unsigned flags, wave_pairs[kWaves];
  const int slots = small_slots(n);
  unsigned* const slot = reinterpret_cast<unsigned*>(keys + (n + 1) / 2 * 2);  // (16-byte aligned)
  const int t = threadIdx.x, lane = t & 63, wib = t >> 6;
  const int share = (rows_pad + gridDim.x - 1) / gridDim.x, first = blockIdx.x * share, last = min(rows_pad, first + share);
  // The upper bits of a hash choose a bucket of four slots, which fill in order and are read at once (single slots: chains of a
  // dozen steps for the slowest lane of a wave, 30 us for 5k rows against 27); the lower 19 stand in the slot.
  const int shift = __clz(slots) + 3, buckets = slots / 4;
  auto place = [&](unsigned h) { return (int)(h >> shift); };
  auto entry = [&](unsigned h, int row) { return (h << kSmallRowBits) | (unsigned)row; };
  if (t == 0) flags = 0;
  for (int i = t; i < slots; i += kSmallThreads) slot[i] = kSmallEmpty;
  constexpr int U = kSmallRows / kSmallThreads;
  unsigned long long mine[U];
  unsigned bad = 0;
  {
    int4 c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = u * kSmallThreads + t < n ? rows[u * kSmallThreads + t] : make_int4(-1, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = u * kSmallThreads + t;
      if (j >= n) {
        mine[u] = kEmpty;
        continue;
      }
      const bool ok = coord_ok(c[u].x, c[u].y, c[u].z, c[u].w);
      mine[u] = ok ? pack_key(c[u].x, c[u].y, c[u].z, c[u].w) : kEmpty;
      if (!ok) bad |= (unsigned)FLAG_RANGE;
      keys[j] = mine[u];
      if (j >= first && j < last) keep[j] = c[u];  // the kmap's own copy of the caller's rows
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (mine[u] == kEmpty) continue;
    const unsigned h = hash_run(mine[u]), e = entry(h, u * kSmallThreads + t);
    int at = place(h);
    bool done = false;
    for (int it = 0; it < buckets && !done; ++it) {
      const uint4 v4 = *reinterpret_cast<const uint4*>(slot + 4 * at);
      const unsigned v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (done) continue;
        unsigned old = v[i];
        if (old == kSmallEmpty) old = atomicCAS(&slot[4 * at + i], kSmallEmpty, e);
        done = old == kSmallEmpty;
        if (!done && ((old ^ e) >> kSmallRowBits) == 0 && keys[old & ((1u << kSmallRowBits) - 1u)] == mine[u]) {
          bad |= (unsigned)FLAG_DUP;
          done = true;
        }
      }
      at = at + 1 == buckets ? 0 : at + 1;
    }
  }
  if (bad) atomicOr(&flags, bad);
  __syncthreads();
  // two rows per wave, a lane per offset
  const int sub = lane / V, k = lane - sub * V;
  const int dx = k / 9 - 1, dy = k / 3 % 3 - 1, dz = k % 3 - 1;
  unsigned pairs = 0;
  for (int r0 = first + wib * RPW; r0 < last; r0 += kWaves * RPW) {
    const int row = r0 + sub;
    const bool active = sub < RPW && row < last;
    int found = -1;
    if (active && row < n && keys[row] != kEmpty) {
      const unsigned long long own = keys[row];
      const int b = (int)(own >> 48), x = (int)((own >> 32) & 0xFFFF) - 32768 + dx, y = (int)((own >> 16) & 0xFFFF) - 32768 + dy,
                z = (int)(own & 0xFFFF) - 32768 + dz;
      if (coord_ok(b, x, y, z)) {
        const unsigned long long key = pack_key(b, x, y, z);
        const unsigned h = hash_run(key), e = entry(h, 0);
        int at = place(h);
        bool done = false;
        for (int it = 0; it < buckets && !done; ++it) {
          const uint4 v4 = *reinterpret_cast<const uint4*>(slot + 4 * at);
          const unsigned v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int j = (int)(v[i] & ((1u << kSmallRowBits) - 1u));
            done = done || v[i] == kSmallEmpty;
            if (!done && ((v[i] ^ e) >> kSmallRowBits) == 0 && keys[j] == key) {
              found = j;
              done = true;
            }
          }
          at = at + 1 == buckets ? 0 : at + 1;
        }
      }
    }
    if (active) map[row * V + k] = found;  // (rows of the padding: no neighbours)
    const unsigned long long bal = __ballot(found >= 0);
    if (active && k == 0) mask[row] = (unsigned)((bal >> (sub * V)) & ((1ull << V) - 1ull));
    pairs += (unsigned)__popcll(bal);
  }
  if (lane == 0) wave_pairs[wib] = pairs;
  __syncthreads();
  if (t == 0) {
    unsigned sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += wave_pairs[w];
    ctl->pairs[blockIdx.x * 16] = sum;
  }
  if (blockIdx.x == 0 && t < kPairSlots) {  // the rest of what k_publish reads (every workgroup has seen every row)
    if (t >= (int)gridDim.x) ctl->pairs[t * 16] = 0;
    ctl->entries[t * 16] = 0;
    ctl->key_or[t * 16] = 0;
    ctl->key_and[t * 16] = 0;
    if (t == 0) {
      ctl->flags = flags;
      ctl->count = 0;
    }
  }
}

// K = 5, submanifold: the 125 offsets as five x-planes of 25 (dx = g - 2; offset j of a plane is
// dy = j / 5 - 2, dz = j % 5 - 2), one map and one 25-bit mask array per plane.  blockIdx.y is the
// plane; five lanes per row, one per column (dx, dy), twelve rows per wave.  A column's five cells z - 2 .. z + 2 lie in
// two runs, so a row takes 50 entry reads in all.  The kernel is bound by the read requests in flight: one lookup
// per offset (125 reads of a table of single voxels) took 102 us at 60k rows of a LiDAR-like scan, this takes
// 40 us; cells 2 and 3 are therefore fetched only where the key matches.
struct Planes5 {
  int* map[5];
  unsigned* mask[5];
};
template <bool FILTER>
__global__ void __launch_bounds__(FILTER ? kProbeThreads : 256)
    k_probe_planes5(const int4* __restrict__ rows, int n_rows, long long rows_pad, const RunSlot* __restrict__ tab, int log_cap,
                    const unsigned* __restrict__ filter_bits, Planes5 pl, Ctl* ctl) {
  constexpr int VP = 25, LPR = 5, RPW = 12, kWaves = FILTER ? kProbeThreads / 64 : 4;
  __shared__ unsigned wave_pairs[kWaves];
  extern __shared__ unsigned filter[];
  const int g = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const long long waves = (long long)gridDim.x * kWaves;
  const int sub = lane / LPR, col = lane - sub * LPR;
  unsigned pairs = 0;
  if constexpr (FILTER) load_filter(filter_bits, filter);
  for (long long wave = (long long)blockIdx.x * kWaves + (threadIdx.x >> 6); wave * RPW < rows_pad; wave += waves) {
    const long long row = wave * RPW + sub;
    const bool active = (sub < RPW) && (row < rows_pad);
    int nb[5] = {-1, -1, -1, -1, -1};
    if (active && row < n_rows) {
      const int4 c = rows[row];
      const int tx = c.y + g - 2, ty = c.z + col - 2;
      if (coord_ok(c.x, c.y, c.z, c.w) && coord_ok(c.x, tx, ty, c.w)) {
        probe_column<FILTER>(c.x, tx, ty, c.w, tab, log_cap, filter, nb);
        // a row that does not find itself at its own place shares it with another row
        if (g == 2 && col == 2 && nb[2] != (int)row) atomicOr(&ctl->flags, FLAG_DUP);
      }
    }
    if (active) {
      int* dst = pl.map[g] + row * VP + LPR * col;
#pragma unroll
      for (int d = 0; d < 5; ++d) dst[d] = nb[d];
    }
    unsigned bits = 0;
#pragma unroll
    for (int d = 0; d < 5; ++d) {
      bits |= (nb[d] >= 0 ? 1u : 0u) << (LPR * col + d);
      pairs += (unsigned)__popcll(__ballot(nb[d] >= 0));
    }
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < LPR; ++i) m |= __shfl(bits, min(lane + i, 63));  // (complete where col == 0)
    if (active && col == 0) pl.mask[g][row] = m;
    if (!FILTER) break;  // (the grid covers the rows)
  }
  if (lane == 0) wave_pairs[threadIdx.x >> 6] = pairs;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned n = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) n += wave_pairs[w];
    if (n) atomicAdd(&ctl->pairs[(g * kPlaneSlots + blockIdx.x % kPlaneSlots) * 16], (unsigned long long)n);
  }
}

// T[j][k] = n for every present pair M[n][k] = j.
__global__ void __launch_bounds__(256) k_scatter_in_side(const int* __restrict__ map, long long n_entries, int V,
                                                         int* __restrict__ tmap) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_entries) return;
  const int j = map[e];
  if (j >= 0) {
    const long long n = e / V;
    const int k = (int)(e - n * V);
    tmap[(long long)j * V + k] = (int)n;
  }
}

// The input side of a stride-2 map from its rows' candidates, every entry and mask in one pass (presets, k_scatter_in_side and
// k_mask_from_map took 6, 8.5 and 7 us at 200k rows).  A workgroup puts the candidates of 64 rows into their places in LDS and writes
// the rows from there (with an address worked out for every entry instead of every candidate: 12 us).
// Along an axis, an even coordinate has offset 0 to the first candidate, an odd one 1 to the first and -1 to the second.
template <int K>
__global__ void __launch_bounds__(256) k_in_side(const int4* __restrict__ rows, const int* __restrict__ cands, long long n_rows,
                                                 uint4* __restrict__ map, unsigned* __restrict__ mask) {
  constexpr int C = cands_of(K), V = K * K * K, R = 64, U = (R * C + 255) / 256;
  __shared__ __align__(16) int s[R * V];
  __shared__ unsigned m[R];
  const int t = threadIdx.x;
  const long long row0 = (long long)blockIdx.x * R;  // (rows_pad is a multiple of 256)
  int c[U];
  int4 p[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const int q = i * 256 + t;
    const bool live = q < R * C && row0 + q / C < n_rows;
    c[i] = live ? cands[row0 * C + q] : -1;
    p[i] = live ? rows[row0 + q / C] : make_int4(0, 0, 0, 0);
  }
  for (int i = t; i < R * V / 4; i += 256) reinterpret_cast<uint4*>(s)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
  if (t < R) m[t] = 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < U; ++i) {
    if (c[i] < 0) continue;
    const int q = i * 256 + t, r = q / C, u = q % C;
    auto digit = [&](int x, int second) { return K == 2 ? x & 1 : x & 1 ? (second ? 0 : 2) : 1; };
    const int k = (digit(p[i].y, u & 4) * K + digit(p[i].z, u & 2)) * K + digit(p[i].w, u & 1);
    s[r * V + k] = c[i];
    atomicOr(&m[r], 1u << k);
  }
  __syncthreads();
  for (int i = t; i < R * V / 4; i += 256) map[row0 * V / 4 + i] = reinterpret_cast<const uint4*>(s)[i];
  if (t < R) mask[row0 + t] = m[t];
}

// Masks of finished map rows.  One load covers two rows of 27 entries; on large maps a wave has eight in flight and
// stores their 16 masks together (200k -> 127k rows and back: 9.5 -> 6.9 us), on small ones the
// waves are few and one load each is quicker (10k to 30k rows: 3.4 us against 5.0).
template <int V, int LOADS> struct MaskRows {
  static constexpr int per_load = 64 / V, loads = LOADS, per_wave = per_load * loads;
  static_assert(per_wave <= 64, "a lane stores the mask of at most one row");
};
template <int V, int LOADS>
__global__ void __launch_bounds__(256) k_mask_from_map(const int* __restrict__ map, int n_rows,
                                                       unsigned* __restrict__ mask, Ctl* ctl, bool counted) {
  if (counted) n_rows = min(n_rows, (int)ctl->count);  // (the launch covers the most rows that there can be)
  __shared__ unsigned wave_cnt[4];
  typedef MaskRows<V, LOADS> R;
  const int lane = threadIdx.x & 63;
  const long long row0 = (((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * R::per_wave;
  const long long left = n_rows - row0;  // rows of this wave (may be <= 0)
  int v[R::loads];
#pragma unroll
  for (int u = 0; u < R::loads; ++u)
    v[u] = lane < R::per_load * V && u * R::per_load + lane / V < left ? map[(row0 + u * R::per_load) * V + lane] : -1;
  unsigned mine = 0, found = 0;
#pragma unroll
  for (int u = 0; u < R::loads; ++u) {
    const unsigned long long bal = __ballot(v[u] >= 0);
    found += (unsigned)__popcll(bal);
    if (lane / R::per_load == u) mine = (unsigned)((bal >> (lane % R::per_load * V)) & ((1ull << V) - 1ull));
  }
  if (lane < R::per_wave && lane < left) mask[row0 + lane] = mine;
  if (!ctl) return;  // (uniform) otherwise count the present entries, one atomic per workgroup
  if (lane == 0) wave_cnt[threadIdx.x >> 6] = found;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned n = wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
    if (n) atomicAdd(&ctl->entries[(blockIdx.x % kPairSlots) * 16], (unsigned long long)n);
  }
}

// The unique coarse keys vary in a few bit ranges only (per 16-bit field: lowest to highest
// varying bit).  Squeezing those ranges together gives a dense key of usually <= 32 bits whose
// order is the order of the full keys, so the sort moves half the bytes in half the passes.
struct BitRuns {
  int n, total;
  int pos[4], len[4], out[4];
  unsigned long long base;  // the constant bits
};
__global__ void __launch_bounds__(256) k_compress_keys(const unsigned long long* __restrict__ keys, int n, BitRuns r,
                                                       unsigned* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const unsigned long long k = keys[i];
  unsigned c = 0;
  for (int j = 0; j < r.n; ++j) c |= (unsigned)((k >> r.pos[j]) & ((1ull << r.len[j]) - 1ull)) << r.out[j];
  out[i] = c;
}
// Sorted dense keys -> coordinates of the coarse points, and each key's rank as its table value.
__global__ void __launch_bounds__(256) k_expand_keys(const unsigned* __restrict__ dense, int n, BitRuns r,
                                                     int4* __restrict__ coords, unsigned long long* tab,
                                                     int log_cap) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const unsigned c = dense[i];
  unsigned long long k = r.base;
  for (int j = 0; j < r.n; ++j) k |= ((unsigned long long)((c >> r.out[j]) & ((1u << r.len[j]) - 1u))) << r.pos[j];
  int4 q;
  q.x = (int)(k >> 48);
  q.y = (int)((k >> 32) & 0xFFFF) - 32768;
  q.z = (int)((k >> 16) & 0xFFFF) - 32768;
  q.w = (int)(k & 0xFFFF) - 32768;
  coords[i] = q;
  if (tab) {
    unsigned slot = 0;
    if (table_find(tab, log_cap, k, &slot) >= 0) tab[2 * (size_t)slot + 1] = (unsigned long long)(unsigned)i;
  }
}

// Per-offset pair counts from the bitmasks.
__global__ void __launch_bounds__(256) k_count_pairs(const unsigned* __restrict__ mask, int n_rows,
                                                     unsigned long long* __restrict__ counts) {
  __shared__ unsigned cnt[32];
  if (threadIdx.x < 32) cnt[threadIdx.x] = 0;
  __syncthreads();
  for (long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x; r < n_rows;
       r += (long long)gridDim.x * blockDim.x) {
    unsigned m = mask[r];
    while (m) {
      const int k = __ffs((int)m) - 1;
      m &= m - 1;
      atomicAdd(&cnt[k], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x < 32 && cnt[threadIdx.x]) atomicAdd(&counts[threadIdx.x], (unsigned long long)cnt[threadIdx.x]);
}

int log2_capacity(int64_t n) {
  int lc = 10;
  while ((1ll << lc) < 2 * n) ++lc;
  return lc;
}

inline unsigned blocks_for(int64_t n, int per_block) { return (unsigned)ceil_div(n > 0 ? n : 1, per_block); }

template <int K>
int launch_probe(bool transposed, const int4* rows, int64_t n_rows, int stride, const unsigned long long* tab,
                 int log_cap, int* map, unsigned* mask, Ctl* ctl, hipStream_t st) {
  constexpr int V = K * K * K;
  constexpr int RPW = 64 / V;
  const int64_t waves = ceil_div(n_rows, RPW);
  const unsigned blocks = blocks_for(waves, 4);
  if (transposed)
    hipLaunchKernelGGL((k_probe<K, true>), dim3(blocks), dim3(256), 0, st, rows, (int)n_rows, stride, tab, log_cap,
                       map, mask, ctl);
  else
    hipLaunchKernelGGL((k_probe<K, false>), dim3(blocks), dim3(256), 0, st, rows, (int)n_rows, stride, tab,
                       log_cap, map, mask, ctl);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

// Presets of a table in one launch: map entries [0, n_map) = -1 (absent), masks [0, n_mask) = 0.
__global__ void __launch_bounds__(256) k_fill_side(unsigned* __restrict__ map, long long n_map, unsigned* __restrict__ mask,
                                                   long long n_mask) {
  const long long stride = (long long)gridDim.x * blockDim.x, t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long long i = t; i < n_map; i += stride) map[i] = 0xFFFFFFFFu;
  for (long long i = t; i < n_mask; i += stride) mask[i] = 0u;
}

int fill_u32(void* dst, int64_t n, unsigned v, hipStream_t st) {
  if (n <= 0) return SPCONV_OK;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)std::min<int64_t>(ceil_div(n, 256), 2048)), dim3(256), 0, st,
                     static_cast<unsigned*>(dst), (long long)n, v);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

// Allocates map and masks; presets the padding rows (no neighbours), or every row when the
// builder only writes the entries that are present.
int alloc_side(SideMap& side, int64_t rows, int V, hipStream_t st, bool preset_all = false) {
  side.rows = rows;
  side.rows_pad = round_up(rows > 0 ? rows : 1, kRowPad);
  SPC_TRY(side.map.alloc((size_t)side.rows_pad * V * sizeof(int)));
  SPC_TRY(side.mask.alloc((size_t)side.rows_pad * sizeof(unsigned)));
  const int64_t first = preset_all ? 0 : rows;
  if (side.rows_pad > first) {
    const int64_t n_map = (side.rows_pad - first) * V;
    hipLaunchKernelGGL(k_fill_side, dim3((unsigned)std::min<int64_t>(ceil_div(n_map, 1024), 2048)), dim3(256), 0, st,
                       side.map.as<unsigned>() + first * V, (long long)n_map, side.mask.as<unsigned>() + first,
                       (long long)(side.rows_pad - first));
    SPC_LAUNCH_CHECK();
  }
  return SPCONV_OK;
}

// Pool of pinned control blocks.  The probe's last workgroup stores the result word; the host finds
// out by reading the word, so nothing is recorded on the stream behind the probe (an event there
// delayed the next kernel by 5.6 us).
struct HostCtl {
  HostResult res;
  HostResult* dev;  // device-side address of res
};

std::mutex g_host_mu;
std::vector<HostCtl*> g_host_free;

HostCtl* host_ctl_acquire() {
  {
    std::lock_guard<std::mutex> lk(g_host_mu);
    if (!g_host_free.empty()) {
      HostCtl* h = g_host_free.back();
      g_host_free.pop_back();
      return h;
    }
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, sizeof(HostCtl), hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  HostCtl* h = static_cast<HostCtl*>(p);
  void* dp = nullptr;
  if (hipHostGetDevicePointer(&dp, p, 0) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipHostFree(p);
    return nullptr;
  }
  h->dev = &static_cast<HostCtl*>(dp)->res;
  return h;
}

// Waits (briefly, yielding) for the result word of a block to be written.
bool host_ctl_ready(const HostCtl* h, double max_seconds) {
  const volatile unsigned long long* w = &h->res.word;
  const auto t0 = std::chrono::steady_clock::now();
  while (!(*w & kHostReady)) {
    const double waited = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (waited > max_seconds) return false;
    if (waited > 2e-4) std::this_thread::yield();
  }
  return true;
}

void host_ctl_release(HostCtl* h) {
  std::lock_guard<std::mutex> lk(g_host_mu);
  g_host_free.push_back(h);
}

// Waits for what the work enqueued on st stores into a block.  launched: what the launches came to.
enum : unsigned { kWaitWord = 1, kWaitOutputs = 2, kWaitReady = 4 };
int wait_block(const HostCtl* hc, unsigned what, hipError_t launched, hipStream_t st) {
  if (launched != hipSuccess) {
    (void)hipStreamSynchronize(st);  // (what was launched may still store)
    return hip_fail(launched, "launch", __FILE__, __LINE__);
  }
  const volatile HostResult* r = &hc->res;
  auto there = [&]() {
    return (!(what & kWaitWord) || (r->word & kHostReady)) && (!(what & kWaitOutputs) || (r->outputs & kHostReady)) &&
           (!(what & kWaitReady) || r->ready);
  };
  const auto t0 = std::chrono::steady_clock::now();
  while (!there()) {  // polled: the work behind it usually takes well under a millisecond
    const double waited = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (waited > 2e-4) std::this_thread::yield();
    if (waited <= 0.01) continue;
    SPC_HIP(hipStreamSynchronize(st));
    if (!there()) return SPCONV_EHIP;
    break;
  }
  std::atomic_thread_fence(std::memory_order_acquire);
  return SPCONV_OK;
}

// Launches k_publish behind the work enqueued so far and waits for its figures.
template <Publish WHAT = kPublishAll> int read_ctl(const Ctl* ctl, HostResult* res, hipStream_t st) {
  HostCtl* hc = host_ctl_acquire();
  if (!hc) return SPCONV_ENOMEM;
  hc->res.word = hc->res.outputs = hc->res.ready = 0;  // (pinned memory: visible to the kernel launched below)
  hipLaunchKernelGGL(k_publish<WHAT>, dim3(1), dim3(64), 0, st, ctl, hc->dev);
  static_assert(WHAT != kPublishWord, "(read by the builds themselves)");
  const int status = wait_block(hc, WHAT == kPublishOutputs ? kWaitWord | kWaitOutputs : kWaitReady, hipGetLastError(), st);
  if (status == SPCONV_OK) {
    *res = hc->res;
    if (WHAT == kPublishOutputs) {
      res->flags = (res->word >> 48) & 0xFFu;
      res->pairs = res->word & 0xFFFFFFFFFFFFull;
      res->count = res->outputs & ~kHostReady;
    }
  }
  host_ctl_release(hc);
  return status;
}

// counted: ctl->count rows, at most `rows`
template <int V> int masks_from_map(const int* map, int64_t rows, unsigned* mask, Ctl* ctl, hipStream_t st, bool counted = false) {
  constexpr int kMany = V == 27 ? 8 : 1;
  auto blocks = [&](int per_wave) { return dim3(blocks_for(ceil_div(rows, per_wave), 4)); };
  if (rows >= 65536)
    hipLaunchKernelGGL((k_mask_from_map<V, kMany>), blocks(MaskRows<V, kMany>::per_wave), dim3(256), 0, st, map, (int)rows, mask, ctl, counted);
  else
    hipLaunchKernelGGL((k_mask_from_map<V, 1>), blocks(MaskRows<V, 1>::per_wave), dim3(256), 0, st, map, (int)rows, mask, ctl, counted);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

int flags_status(unsigned long long flags) {
  if (flags & FLAG_RANGE) return SPCONV_ERANGE;
  if (flags & FLAG_DUP) return SPCONV_EDUP;
  if (flags & FLAG_FULL) return SPCONV_ENOMEM;
  return SPCONV_OK;
}


int build_init(const DevBuf& tab, long long words /*of 16 bytes*/, Ctl* ctl, hipStream_t st, int marks = 0) {
  hipLaunchKernelGGL(k_build_init, dim3((unsigned)std::min<int64_t>(ceil_div(words, 256), 4096)), dim3(256), 0, st,
                     tab.as<ulonglong2>(), words, marks, ctl);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

// The table of z-runs of a 5x5x5 build, and from a number of rows on the probe's filter.  Whole waited builds without and with it, us:
//   scan 20k rows 50, 52; 50k 72, 71; 80k 93, 80; 120k 134, 113; room 20k 47, 48; 50k 65, 65; 80k 90, 82; uniform 50k 79, 78.5; 80k 106, 92
// (In buckets, as 3x3x3 builds are, a row has 2.5 times the copies and 2.8 times the look-ups: 9k rows of a scan 29, 35; 30k 51,
// 50; 60k 67, 60 to 72; 80k 67, 75 to 80: neither is ahead.)
struct RunTable {
  DevBuf buf;  // entries, then (with a filter) its marks and its bits
  int log_cap = 0;
  unsigned char* marks = nullptr;
  unsigned* bits = nullptr;
};
constexpr int64_t kFilterRows5 = 50000;
int build_runs(const int4* rows, int64_t N, bool filter, Ctl* ctl, int4* keep, RunTable* t, hipStream_t st) {
  t->log_cap = log2_capacity(N);  // entries >= 2 N >= twice the z-runs
  const size_t table = sizeof(RunSlot) << t->log_cap;
  SPC_TRY(t->buf.alloc(table + (filter ? ((size_t)1 << kFilterBits) + kFilterWords * 4 : 0)));
  if (filter) {
    t->marks = t->buf.as<unsigned char>() + table;
    t->bits = reinterpret_cast<unsigned*>(t->marks + ((size_t)1 << kFilterBits));
  }
  SPC_TRY(build_init(t->buf, 2ll << t->log_cap, ctl, st, filter ? kMarkWords : 0));
  hipLaunchKernelGGL(k_insert_runs, dim3(blocks_for(N, 256)), dim3(256), 0, st, rows, (int)N, t->buf.as<RunSlot>(), t->log_cap,
                     ctl, keep, t->marks);
  SPC_LAUNCH_CHECK();
  if (!filter) return SPCONV_OK;
  hipLaunchKernelGGL(k_filter_pack, dim3(kFilterWords / 256), dim3(256), 0, st, reinterpret_cast<const uint4*>(t->marks), t->bits);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}
template <typename F> int allow_lds(F kernel, int bytes, std::atomic<bool>& done) {  // (set twice by racing threads at worst)
  if (done.load(std::memory_order_acquire)) return SPCONV_OK;
  SPC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
  done.store(true, std::memory_order_release);
  return SPCONV_OK;
}

// The buckets of a submanifold 3x3x3 build.  Up to 512, of 64 rows at least: they all run at once; from then on 256 rows a bucket,
// which weighs a workgroup's fixed 5 us against the longest bucket (us, with 128, 256 rows a bucket: 60k rows of a scan 23, 28; of a room 26, 35;
// 100k 30, 26; 400k 82, 67; with 350: buckets beyond kBucketRows, 300k of a room 83 against 64).  There are 2^kMaxBucketBits of them at
// most, whose counts are what a dealer holds in LDS.  Where they would have more than 512 rows (with the copies up to kBucketRows, and
// beyond that look-ups once per round), the rows are dealt in parts, each a dealing and a look-up launch over its share of the buckets.
// Waited builds with a table of runs in memory, in rounds, in parts, ms: 8M rows, 15 % of the cells of their box 3.6, 1.6, 1.6; 16M 7.9, 5.0,
// 3.6; 40M 22, 31, 15; 0.2 % 4.9, 1.4, 1.4; 10.5, 7.0, 3.1; 23, 42, 13.
struct Buckets {
  int dealers, per, log_b = 6, log_parts = 0;
  size_t entries, starts, bytes;
  explicit Buckets(int64_t N) {
    per = (int)std::max<int64_t>(round_up(ceil_div(N, kDealers), kDealThreads), kDealThreads);
    dealers = (int)ceil_div(N, per);
    while (log_b < kMaxBucketBits && (log_b < 9 ? (int64_t)64 << log_b : (int64_t)256 << log_b) < N) ++log_b;
    while (((int64_t)512 << (kMaxBucketBits + log_parts)) < N) ++log_parts;
    entries = (size_t)dealers * per * kCopies * sizeof(Dealt);
    starts = (size_t)dealers * ((2 << log_b) + 1) * sizeof(unsigned);
    bytes = entries + starts + (size_t)dealers * sizeof(unsigned);
  }
};

// Submanifold 3x3x3 build: rows into buckets, look-ups (whose last workgroup publishes the result to
// pinned host memory); small maps: one launch, and k_publish.  kRetryTable where there is no memory for the buckets (about 100 bytes a
// row, room for a row in eight of them; a table of single rows takes 32 to 64).
int build_submanifold3(spconv_kmap* km, const int4* rows, int64_t N, bool async, hipStream_t st) {
  const int V = 27;
  DevBuf ctl_buf, own_rows, dealt;
  SPC_TRY(ctl_buf.alloc(sizeof(Ctl)));
  Ctl* ctl = ctl_buf.as<Ctl>();
  const bool small = N <= kSmallRows;
  const Buckets bk(N);
  const int small_lds = (int)round_up(N, 2) * 8 + small_slots((int)std::min<int64_t>(N, kSmallRows)) * 4;
  static std::atomic<bool> deal_lds_set{false}, deal_parts_lds_set{false}, small_lds_set{false};
  if (small) SPC_TRY(allow_lds(k_build_small3, kSmallRows * 8 + small_slots(kSmallRows) * 4, small_lds_set));
  else if (bk.log_parts) SPC_TRY(allow_lds(k_deal_rows<true>, deal_lds(kMaxBucketBits), deal_parts_lds_set));
  else SPC_TRY(allow_lds(k_deal_rows<false>, deal_lds(kMaxBucketBits), deal_lds_set));
  SPC_TRY(own_rows.alloc((size_t)N * 16));
  SideMap& side = km->out_side;
  side.rows = N;
  side.rows_pad = round_up(N, kRowPad);
  SPC_TRY(side.map.alloc((size_t)side.rows_pad * V * sizeof(int)));
  SPC_TRY(side.mask.alloc((size_t)side.rows_pad * sizeof(unsigned)));
  if (!small && dealt.alloc(bk.bytes) != SPCONV_OK) return capturing(st) ? SPCONV_ENOMEM : kRetryTable;  // (that build waits)
  HostCtl* hc = host_ctl_acquire();
  if (!hc) return SPCONV_ENOMEM;
  hc->res.word = hc->res.ready = 0;  // (pinned memory: visible to the kernels launched below)
  if (small)
    hipLaunchKernelGGL(k_build_small3, dim3((unsigned)std::min<int64_t>(ceil_div(side.rows_pad, 32), kSmallWgs)), dim3(kSmallThreads),
                       small_lds, st, rows, (int)N, (int)side.rows_pad, own_rows.as<int4>(), side.map.as<int>(),
                       side.mask.as<unsigned>(), ctl);
  else {
    Dealt* const entries = dealt.as<Dealt>();
    unsigned* const starts = reinterpret_cast<unsigned*>(dealt.as<char>() + bk.entries);
    unsigned* const flags = reinterpret_cast<unsigned*>(dealt.as<char>() + bk.entries + bk.starts);
    const unsigned parts = 1u << bk.log_parts;
    for (unsigned part = 0; part < parts; ++part) {
      hipLaunchKernelGGL(parts > 1 ? k_deal_rows<true> : k_deal_rows<false>, dim3((unsigned)bk.dealers), dim3(kDealThreads), deal_lds(bk.log_b), st, rows, (int)N, bk.per, bk.log_b,
                         bk.log_parts, part, entries, starts, flags, own_rows.as<int4>(), (long long)side.rows_pad, side.map.as<int>(),
                         side.mask.as<unsigned>(), ctl);
      hipLaunchKernelGGL(k_probe_buckets, dim3(1u << bk.log_b), dim3(kBucketThreads), 0, st, entries, starts, flags, bk.dealers, bk.per,
                         bk.log_b, parts, side.map.as<int>(), side.mask.as<unsigned>(), ctl, hc->dev);
    }
  }
  // (a waited build: a kernel of its own reports the end, and once it runs, the stores before it are visible to every stream)
  if (small) hipLaunchKernelGGL(k_publish<kPublishWord>, dim3(1), dim3(64), 0, st, ctl, hc->dev);
  else if (!async) hipLaunchKernelGGL(k_publish<kPublishEnd>, dim3(1), dim3(64), 0, st, ctl, hc->dev);
  const bool ok = hipGetLastError() == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    (void)hipStreamSynchronize(st);
    host_ctl_release(hc);
    return SPCONV_EHIP;
  }
  km->n_in = km->n_out = N;
  side.ready = true;
  km->pending_host = hc;
  km->pending = true;
  km->n_pairs = -1;
  // (ctl_buf returns to the pool here; reuse is ordered behind the probe on this stream)
  if (!async) {
    const int rc = wait_block(hc, small ? kWaitWord : kWaitWord | kWaitReady, hipSuccess, st);
    const unsigned long long word = hc->res.word;
    km->pending = false;
    km->pending_host = nullptr;
    if (rc != SPCONV_OK) (void)hipStreamSynchronize(st);  // (the probe still writes to hc)
    host_ctl_release(hc);
    SPC_TRY(rc);
    km->n_pairs = (int64_t)(word & 0xFFFFFFFFFFFFull);
    km->build_status = flags_status((word >> 48) & 0xFFu);
    SPC_TRY(km->build_status);
  }
  std::swap(km->in_coords.p, own_rows.p);  // P_out == P_in: out_coords stays empty
  std::swap(km->in_coords.bytes, own_rows.bytes);
  return SPCONV_OK;
}

// K = 5 submanifold build: one table of the rows, one probe launch over the five planes, one read of
// the control block (flags and the planes' pair counts).
int build_submanifold5(spconv_kmap* km, const int4* rows, int64_t N, hipStream_t st) {
  constexpr int VP = 25;
  DevBuf ctl_buf, own_rows;
  RunTable tab;
  SPC_TRY(ctl_buf.alloc(sizeof(Ctl)));
  Ctl* ctl = ctl_buf.as<Ctl>();
  const bool filter = N >= kFilterRows5;
  static std::atomic<bool> lds_allowed{false};
  if (filter) SPC_TRY(allow_lds(k_probe_planes5<true>, kFilterWords * 4, lds_allowed));
  SPC_TRY(own_rows.alloc((size_t)N * 16));
  SPC_TRY(build_runs(rows, N, filter, ctl, own_rows.as<int4>(), &tab, st));
  Planes5 pl{};
  for (int g = 0; g < 5; ++g) {
    std::unique_ptr<spconv_kmap> sub(new (std::nothrow) spconv_kmap(
        std::make_shared<SideMap>(), std::make_shared<SideMap>(), km->in_coords_ref, km->out_coords_ref));
    if (!sub) return SPCONV_ENOMEM;
    sub->K = 5;
    sub->V = VP;
    sub->n_in = sub->n_out = N;
    sub->build_stream = sub->last_stream = st;
    sub->out_side.rows = N;
    sub->out_side.rows_pad = round_up(N, kRowPad);
    SPC_TRY(sub->out_side.map.alloc((size_t)sub->out_side.rows_pad * VP * sizeof(int)));  // (padding rows are the probe's)
    SPC_TRY(sub->out_side.mask.alloc((size_t)sub->out_side.rows_pad * sizeof(unsigned)));
    sub->out_side.ready = true;
    pl.map[g] = sub->out_side.map.as<int>();
    pl.mask[g] = sub->out_side.mask.as<unsigned>();
    km->groups.push_back(std::move(sub));
  }
  const long long rows_pad = round_up(N, kRowPad);
  if (filter)
    hipLaunchKernelGGL(k_probe_planes5<true>, dim3(51, 5), dim3(kProbeThreads), kFilterWords * 4, st, rows, (int)N, rows_pad,
                       tab.buf.as<RunSlot>(), tab.log_cap, tab.bits, pl, ctl);
  else
    hipLaunchKernelGGL(k_probe_planes5<false>, dim3(blocks_for(ceil_div(rows_pad, 12), 4), 5), dim3(256), 0, st, rows, (int)N, rows_pad,
                       tab.buf.as<RunSlot>(), tab.log_cap, (const unsigned*)nullptr, pl, ctl);
  SPC_LAUNCH_CHECK();
  HostResult h{};
  SPC_TRY(read_ctl(ctl, &h, st));
  std::swap(km->in_coords.p, own_rows.p);  // P_out == P_in: out_coords stays empty
  std::swap(km->in_coords.bytes, own_rows.bytes);
  km->n_in = km->n_out = N;
  km->n_pairs = 0;
  for (int g = 0; g < 5; ++g) {
    km->groups[g]->n_pairs = (int64_t)h.plane_pairs[g];
    km->n_pairs += (int64_t)h.plane_pairs[g];
  }
  km->build_status = flags_status(h.flags);
  return km->build_status;
}

// The tables of a stride-2 build are made for as many outputs as inputs, and the kmap keeps them.  Where more than half of that is
// unused, and more than kKeepBytes of it, the used part moves into buffers of its own size: 300k rows of a room, 75k outputs,
// 38 MB -> 10 MB, the build 80 -> 107 us (copy 4 us, the rest is a second wait: smaller surpluses are left: 60k rows 51 -> 82).
// Without memory for the copy everything stays where it is.
constexpr int64_t kKeepBytes = 16 << 20;
int shrink_to_outputs(SideMap& side, int V, DevBuf& coarse_rows, const Ctl* ctl, hipStream_t st) {
  const size_t used[3] = {(size_t)side.rows_pad * V * sizeof(int), (size_t)side.rows_pad * sizeof(unsigned), (size_t)side.rows * 16};
  DevBuf* const from[3] = {&side.map, &side.mask, &coarse_rows};
  size_t all = 0, need = 0;
  for (int a = 0; a < 3; ++a) all += from[a]->bytes, need += used[a];
  if (2 * need >= all || all - need <= (size_t)kKeepBytes) return SPCONV_OK;
  DevBuf to[3];
  Copy3 c{};
  for (int a = 0; a < 3; ++a) {
    if (to[a].alloc(used[a]) != SPCONV_OK) return SPCONV_OK;
    c.src[a] = from[a]->as<uint4>();
    c.dst[a] = to[a].as<uint4>();
    c.words[a] = (long long)(used[a] / 16);
  }
  hipLaunchKernelGGL(k_copy3, dim3((unsigned)std::min<int64_t>(ceil_div((int64_t)(used[0] / 16), 1024), 2048)), dim3(256), 0, st, c);
  SPC_LAUNCH_CHECK();
  for (int a = 0; a < 3; ++a) {  // (the old ones go back to the pool of this stream)
    std::swap(from[a]->p, to[a].p);
    std::swap(from[a]->bytes, to[a].bytes);
  }
  HostResult again{};  // (a build that is waited for is complete when it returns)
  return read_ctl<kPublishEnd>(ctl, &again, st);
}

// What a stride-2 build over the box leaves where the box is too large: the caller's rows, the hash table of the coarse points and
// their keys, an empty table for the fine points behind it (K = 2), and the control block of all this.
struct CoarseTable {
  DevBuf ctl, rows, slots, keys;  // slots: 2^log_cap of the coarse points, as many for the fine ones
  int log_cap = 0;                // 0: nothing is there
};

// Stride-2 builds (K = 2, 3) over a bit per cell of the coarse points' box; kRetryTable where the box is too large (with what the
// table needs, see CoarseTable), or the memory does not suffice: up to 512 bytes a row for bits and prefixes, else two thirds of that
// for boxes of two thirds as many cells (a scan's has a fifth), and tables for N outputs.  The hash table and tables for the outputs
// that there are need less.
int build_down2(spconv_kmap* km, const int4* rows, int64_t N, int K, hipStream_t st, CoarseTable* fallback) {
  const int V = K * K * K;
  int64_t max_words = std::min<int64_t>(std::max<int64_t>(N * (kCellsPerRow / 32), 1 << 15), kMaxBoxWords);
  // about 400 rows to a chunk; dealers of 512 rows and more
  int log_chunks = 6;
  while ((1 << log_chunks) < kMaxChunks && ((int64_t)400 << log_chunks) < N) ++log_chunks;
  const int chunks = 1 << log_chunks;
  const int per = (int)std::max<int64_t>(round_up(ceil_div(N, kBoxDealers), kBoxDealThreads), kBoxDealThreads);
  const int dealers = (int)ceil_div(N, per);
  DevBuf coarse_rows, small, cands;
  DevBuf &ctl_buf = fallback->ctl, &own_rows = fallback->rows, &cells = fallback->slots, &keys = fallback->keys;
  // sized for as many outputs as inputs: their number is read at the end
  SideMap& side = km->out_side;
  const int64_t most = round_up(N, kRowPad);
  const size_t base_bytes = most_groups(chunks) * sizeof(unsigned), partial_bytes = (size_t)kBoxBlocks * 9 * sizeof(int);
  auto buffers = [&]() {
    SPC_TRY(ctl_buf.alloc(sizeof(Ctl)));
    SPC_TRY(own_rows.alloc((size_t)N * 16));
    SPC_TRY(coarse_rows.alloc((size_t)N * 16));
    SPC_TRY(small.alloc(base_bytes + sizeof(Box) + partial_bytes + ((size_t)chunks + (size_t)dealers * (chunks * kMaxWindows + 1)) * sizeof(unsigned)));
    SPC_TRY(cells.alloc((size_t)max_words * sizeof(Cells)));
    SPC_TRY(keys.alloc((size_t)N * 8));
    SPC_TRY(side.map.alloc((size_t)most * V * sizeof(int)));
    return side.mask.alloc((size_t)most * sizeof(unsigned));
  };
  if (buffers() != SPCONV_OK) {
    max_words = max_words * 2 / 3 / 4 * 4;
    for (DevBuf* b : {&cells, &side.map, &side.mask}) b->release();
    if (buffers() != SPCONV_OK) return kRetryTable;
  }
  Ctl* ctl = ctl_buf.as<Ctl>();
  // (two tables in the place of the cells, the keys in that of the rows' cells: too large from two million rows on)
  const int table_cap = log2_capacity(N);
  const long long table_slots = (K == 2 ? 2ll : 1ll) << table_cap;
  const bool table_fits = table_slots * 16 <= max_words * 8 / 2;
  unsigned* base = small.as<unsigned>();
  Box* box = reinterpret_cast<Box*>(small.as<char>() + base_bytes);
  int* partial = reinterpret_cast<int*>(box + 1);
  unsigned *totals = reinterpret_cast<unsigned*>(partial) + kBoxBlocks * 9, *starts = totals + chunks;
  int* map = side.map.as<int>();
  const unsigned n_partial = (unsigned)std::min<int64_t>(ceil_div(N, 1024), kBoxBlocks);
  HostCtl* hc = host_ctl_acquire();
  if (!hc) return SPCONV_ENOMEM;
  hc->res.word = 0;  // (pinned memory: visible to the kernels launched below)
  hipError_t launched = hipSuccess;
  auto check = [&]() {
    const hipError_t e = hipGetLastError();
    if (launched == hipSuccess) launched = e;
  };
  // The box's verdict is there once the second launch has run.  It is waited for where the host is ahead of the GPU anyway: small
  // builds are as fast as their launches (2k rows 57 us, with the wait behind the marks 60).
  bool too_large = false;
  auto verdict = [&]() -> int {
    const int status = wait_block(hc, kWaitWord, launched, st);
    const unsigned long long word = hc->res.word;
    host_ctl_release(hc);
    SPC_TRY(status);
    too_large = (word >> 48) & FLAG_BOX;
    return SPCONV_OK;
  };
  const bool early = N >= 16384;
  hipLaunchKernelGGL(k_box_bounds, dim3(n_partial), dim3(256), 0, st, rows, (int)N, own_rows.as<int4>(), partial);
  check();
  hipLaunchKernelGGL(k_box_deal, dim3((unsigned)dealers), dim3(kBoxDealThreads), 0, st, partial, (int)n_partial, (long long)max_words, rows,
                     (int)N, per, log_chunks, keys.as<unsigned>(), starts, cells.as<ulonglong2>(), table_fits ? table_slots : 0ll, box, ctl,
                     hc->dev);
  check();
  hipLaunchKernelGGL(k_box_bits, dim3((unsigned)chunks), dim3(kBitsThreads), 0, st, box, keys.as<unsigned>(), starts, dealers, per,
                     log_chunks, cells.as<Cells>(), base, totals, rows, (int)N, table_fits ? table_cap : 0, cells.as<unsigned long long>(),
                     keys.as<unsigned long long>(), ctl);
  check();
  if (early) SPC_TRY(verdict());
  if (!too_large) {
    hipLaunchKernelGGL(k_box_base, dim3(1 + (unsigned)std::min<int64_t>(ceil_div(N * V, 16384), 512)), dim3(kBaseThreads), 0, st, box, totals,
                       chunks, base, V, side.map.as<uint4>(), side.mask.as<unsigned>(), ctl);
    check();
    if (!early) SPC_TRY(verdict());
  }
  if (too_large) {
    fallback->log_cap = table_fits ? table_cap : 0;
    return kRetryTable;
  }
  SPC_HIP(launched);
  (void)cands.alloc((size_t)N * cands_of(K) * sizeof(int));  // (done without where there is no room)
  const dim3 scatter_grid(blocks_for(K == 3 ? N * 8 : N, 256));
  if (K == 3)
    hipLaunchKernelGGL(k_box_scatter<3>, scatter_grid, dim3(256), 0, st, rows, (int)N, box, cells.as<Cells>(), base, map, coarse_rows.as<int4>(),
                       cands.as<int>(), ctl);
  else
    hipLaunchKernelGGL(k_box_scatter<2>, scatter_grid, dim3(256), 0, st, rows, (int)N, box, cells.as<Cells>(), base, map, coarse_rows.as<int4>(),
                       cands.as<int>(), ctl);
  SPC_LAUNCH_CHECK();
  SPC_TRY(K == 3 ? masks_from_map<27>(map, N, side.mask.as<unsigned>(), ctl, st, true)
                 : masks_from_map<8>(map, N, side.mask.as<unsigned>(), ctl, st, true));
  HostResult h{};
  SPC_TRY(read_ctl<kPublishOutputs>(ctl, &h, st));
  SPC_TRY(flags_status(h.flags));
  km->n_in = N;
  km->n_out = side.rows = (int64_t)h.count;
  side.rows_pad = round_up(side.rows, kRowPad);
  side.ready = true;
  km->n_pairs = (int64_t)h.pairs;
  SPC_TRY(shrink_to_outputs(side, V, coarse_rows, ctl, st));
  if (cands.p && cands.bytes <= (size_t)side.rows * V * sizeof(int)) {
    std::swap(km->in_side.cands.p, cands.p);
    std::swap(km->in_side.cands.bytes, cands.bytes);
  }
  std::swap(km->in_coords.p, own_rows.p);
  std::swap(km->in_coords.bytes, own_rows.bytes);
  std::swap(km->out_coords.p, coarse_rows.p);
  std::swap(km->out_coords.bytes, coarse_rows.bytes);
  return SPCONV_OK;
}

}  // namespace

struct HostCtlHandle {
  // the probe must have written the block before it is handed to another build
  static void finish(void* p) {
    HostCtl* hc = static_cast<HostCtl*>(p);
    if (!host_ctl_ready(hc, 0.05)) (void)hipDeviceSynchronize();
    host_ctl_release(hc);
  }
};

int kmap_status(spconv_kmap* km, hipStream_t) {
  if (!km->pending) return km->build_status;
  HostCtl* hc = static_cast<HostCtl*>(km->pending_host);
  if (!host_ctl_ready(hc, 0.002)) {
    // not there yet: wait for the stream the build runs on instead of spinning
    SPC_HIP(hipStreamSynchronize(km->build_stream));
  }
  if (!host_ctl_ready(hc, 1.0)) {  // the probe never ran to its end
    (void)hipDeviceSynchronize();
    km->pending = false;
    km->pending_host = nullptr;
    host_ctl_release(hc);
    km->build_status = SPCONV_EHIP;
    return SPCONV_EHIP;
  }
  const unsigned long long word = hc->res.word;
  const int status = flags_status((word >> 48) & 0xFFu);
  km->n_pairs = (int64_t)(word & 0xFFFFFFFFFFFFull);
  km->pending = false;
  km->pending_host = nullptr;
  host_ctl_release(hc);
  km->build_status = status;  // kept: whoever resolved the build (a pair count, a tuner), spconv_kmap_status still reports it
  return status;
}

namespace {
int kmap_build_impl(const int32_t* coords, int64_t N, int K, int stride, int transposed, bool async, hipStream_t st,
                    spconv_kmap** out, bool dilate, bool bit_per_cell, bool few_launch_sort);
}
int kmap_build(const int32_t* coords, int64_t N, int K, int stride, int transposed, bool async, hipStream_t st,
               spconv_kmap** out, bool dilate) {
  int status = kmap_build_impl(coords, N, K, stride, transposed, async, st, out, dilate, true, true);
  if (status == kRetryGeneralSort) status = kmap_build_impl(coords, N, K, stride, transposed, async, st, out, dilate, false, false);
  return status;
}
namespace {
int kmap_build_impl(const int32_t* coords, int64_t N, int K, int stride, int transposed, bool async, hipStream_t st,
                    spconv_kmap** out, bool dilate, bool bit_per_cell, bool few_launch_sort) {
  std::unique_ptr<spconv_kmap> km(new (std::nothrow) spconv_kmap);
  if (!km) return SPCONV_ENOMEM;
  km->K = K;
  km->V = K * K * K;
  km->stride = stride;
  km->transposed = transposed;
  km->dilated = dilate ? 1 : 0;
  km->build_stream = st;
  km->last_stream = st;
  const int V = km->V;
  // builds whose output (or, transposed, input) set is derived from the caller's rows: the coarse
  // points of a strided map, or the dilated set of a stride-1 map
  const bool needs_coarse = stride > 1 || dilate;
  const int64_t cand = dilate ? N * V : N;  // most points that derivation can yield

  if (N == 0) {
    km->n_in = km->n_out = 0;
    km->n_pairs = 0;
    SPC_TRY(km->in_coords.alloc(16));
    SPC_TRY(km->out_coords.alloc(16));
    SPC_TRY(alloc_side(km->out_side, 0, V, st));
    km->out_side.ready = true;
    *out = km.release();
    return SPCONV_OK;
  }

  const int4* rows = reinterpret_cast<const int4*>(coords);
  if (K == 5) {  // (submanifold only: the entry points refuse other K = 5 maps)
    SPC_TRY(build_submanifold5(km.get(), rows, N, st));  // (range and duplicate errors: no kmap, as for every synchronous build)
    *out = km.release();
    return SPCONV_OK;
  }
  if (K == 3 && stride == 1 && !transposed && !dilate) {
    const int status = build_submanifold3(km.get(), rows, N, async, st);
    if (status != kRetryTable) {
      SPC_TRY(status);
      *out = km.release();
      return SPCONV_OK;
    }
  }
  CoarseTable made;  // (log_cap 0: nothing of it)
  if (stride == 2 && (K == 2 || K == 3) && !transposed && bit_per_cell) {
    const int status = build_down2(km.get(), rows, N, K, st, &made);
    if (status != kRetryTable) {
      SPC_TRY(status);
      *out = km.release();
      return SPCONV_OK;
    }
    km->out_side.map.release();
    km->out_side.mask.release();
    if (!made.log_cap)
      for (DevBuf* b : {&made.ctl, &made.rows, &made.slots, &made.keys}) b->release();
  }
  const bool have_table = made.log_cap > 0;
  auto take = [](DevBuf& to, DevBuf& from) {
    std::swap(to.p, from.p);
    std::swap(to.bytes, from.bytes);
  };
  DevBuf ctl_buf, tab_fine, tab_coarse, ukeys_a, ukeys_b, hist;
  if (have_table) {
    take(ctl_buf, made.ctl);
    take(tab_coarse, made.slots);
    take(ukeys_a, made.keys);
  } else {
    SPC_TRY(ctl_buf.alloc(sizeof(Ctl)));
  }
  Ctl* ctl = ctl_buf.as<Ctl>();

  // Stride-2 3x3x3 maps are built from the input side and need no table of the fine points.  (Only
  // stride 2: there every input row meets the output floor(p/2), so every row writes at least one
  // entry and duplicate rows cannot escape the entry count; at larger strides some rows write none.)
  const bool from_inputs = (K == 3 && stride == 2 && !transposed && !dilate);
  // fine table: key(p_j) -> j.  Also the duplicate / range check of the caller's rows.
  const int lc_fine = log2_capacity(N);
  // the caller's rows are kept: they are P_in (and P_out for stride 1), or the fine output set
  DevBuf own_rows;
  if (have_table)
    take(own_rows, made.rows);
  else
    SPC_TRY(own_rows.alloc((size_t)N * 16));
  unsigned long long* fine = nullptr;
  if (!from_inputs) {
    if (have_table) {
      fine = tab_coarse.as<unsigned long long>() + (2ll << made.log_cap);
    } else {
      SPC_TRY(tab_fine.alloc((size_t)16 << lc_fine));
      SPC_TRY(build_init(tab_fine, 1ll << lc_fine, ctl, st));
      fine = tab_fine.as<unsigned long long>();
    }
    hipLaunchKernelGGL(k_insert_rows, dim3(blocks_for(N, 256)), dim3(256), 0, st, rows, (int)N, fine, lc_fine, ctl, own_rows.as<int4>());
    SPC_LAUNCH_CHECK();
  }

  HostResult h{};
  int64_t U = 0;
  DevBuf coarse_rows;
  const int lc_coarse = dilate ? log2_capacity(cand) : lc_fine;
  if (needs_coarse && have_table) {
    SPC_TRY(ukeys_b.alloc((size_t)cand * 8));
  } else if (needs_coarse) {
    SPC_TRY(tab_coarse.alloc((size_t)16 << lc_coarse));
    if (from_inputs)
      SPC_TRY(build_init(tab_coarse, 1ll << lc_coarse, ctl, st));
    else
      SPC_TRY(fill_u32(tab_coarse.p, (int64_t)4 << lc_coarse, 0xFFFFFFFFu, st));
    SPC_TRY(ukeys_a.alloc((size_t)cand * 8));
    SPC_TRY(ukeys_b.alloc((size_t)cand * 8));
    if (dilate) {
      const unsigned blocks = blocks_for(cand, 256);
      if (K == 3)
        hipLaunchKernelGGL(k_dilate_unique<3>, dim3(blocks), dim3(256), 0, st, rows, (long long)N,
                           tab_coarse.as<unsigned long long>(), lc_coarse, ukeys_a.as<unsigned long long>(), ctl);
      else
        hipLaunchKernelGGL(k_dilate_unique<1>, dim3(blocks), dim3(256), 0, st, rows, (long long)N,
                           tab_coarse.as<unsigned long long>(), lc_coarse, ukeys_a.as<unsigned long long>(), ctl);
    } else {
      hipLaunchKernelGGL(k_coarse_unique, dim3(blocks_for(N, 256)), dim3(256), 0, st, rows, (int)N, stride,
                         tab_coarse.as<unsigned long long>(), lc_coarse, ukeys_a.as<unsigned long long>(), ctl,
                         from_inputs ? own_rows.as<int4>() : nullptr);
    }
    SPC_LAUNCH_CHECK();
  }
  if (needs_coarse) {
    // the one synchronisation of a strided build: error flags, U, varying key bits
    SPC_TRY(read_ctl(ctl, &h, st));
    SPC_TRY(flags_status(h.flags));
    U = (int64_t)h.count;
    SPC_TRY(hist.alloc(sort_hist_elems(U) * sizeof(uint32_t)));
    int in_b = 0;
    const unsigned long long varying = h.key_or ^ h.key_and;
    BitRuns runs{};
    runs.base = h.key_and & ~varying;
    for (int f = 0; f < 4; ++f) {
      const unsigned v = (unsigned)((varying >> (16 * f)) & 0xFFFFu);
      if (!v) continue;
      int lo = 0, hi = 15;
      while (!((v >> lo) & 1u)) ++lo;
      while (!((v >> hi) & 1u)) --hi;
      runs.pos[runs.n] = 16 * f + lo;
      runs.len[runs.n] = hi - lo + 1;
      runs.out[runs.n] = runs.total;
      runs.total += hi - lo + 1;
      // (bits inside a span that do not vary travel with the dense key; base must not repeat them)
      runs.base &= ~(((1ull << (hi - lo + 1)) - 1ull) << (16 * f + lo));
      ++runs.n;
    }
    SPC_TRY(coarse_rows.alloc((size_t)U * 16));
    const bool want_rank = transposed || from_inputs;
    if (runs.total <= 32) {
      // ukeys_b's N * 8 bytes hold both dense key buffers
      uint32_t* dense_a = ukeys_b.as<uint32_t>();
      uint32_t* dense_b = dense_a + cand;
      hipLaunchKernelGGL(k_compress_keys, dim3(blocks_for(U, 256)), dim3(256), 0, st,
                         ukeys_a.as<unsigned long long>(), (int)U, runs, dense_a);
      SPC_LAUNCH_CHECK();
      // Builds that read the control block once more at their end (stride-2 3x3x3) sort with one
      // launch per digit; should one of its bounded waits run out, that read shows it and the
      // build is done again with the general sort.
      int sorted = SPCONV_EINVAL;
      if (few_launch_sort && from_inputs)
        sorted = msort_keys_u32(dense_a, dense_b, U, runs.total, reinterpret_cast<unsigned*>(&ctl->flags),
                                (unsigned)FLAG_SORT, st, &in_b);
      if (sorted == SPCONV_EINVAL)
        sorted = radix_sort_u32(dense_a, dense_b, nullptr, nullptr, U, runs.total, hist.as<uint32_t>(), st, &in_b);
      SPC_TRY(sorted);
      hipLaunchKernelGGL(k_expand_keys, dim3(blocks_for(U, 256)), dim3(256), 0, st, in_b ? dense_b : dense_a, (int)U,
                         runs, coarse_rows.as<int4>(),
                         want_rank ? tab_coarse.as<unsigned long long>() : (unsigned long long*)nullptr, lc_coarse);
      SPC_LAUNCH_CHECK();
    } else {
      SPC_TRY(radix_sort_u64(ukeys_a.as<uint64_t>(), ukeys_b.as<uint64_t>(), U, varying, hist.as<uint32_t>(), st,
                             &in_b));
      const unsigned long long* sorted = in_b ? ukeys_b.as<unsigned long long>() : ukeys_a.as<unsigned long long>();
      hipLaunchKernelGGL(k_decode_keys, dim3(blocks_for(U, 256)), dim3(256), 0, st, sorted, (int)U,
                         coarse_rows.as<int4>());
      SPC_LAUNCH_CHECK();
      if (want_rank) {
        hipLaunchKernelGGL(k_assign_rank, dim3(blocks_for(U, 256)), dim3(256), 0, st, sorted, (int)U,
                           tab_coarse.as<unsigned long long>(), lc_coarse);
        SPC_LAUNCH_CHECK();
      }
    }
  }

  int status = SPCONV_OK;
  if (from_inputs) {
    km->n_in = N;
    km->n_out = U;
    SPC_TRY(alloc_side(km->out_side, U, V, st, true));
    hipLaunchKernelGGL(k_scatter_down3, dim3(blocks_for(ceil_div(N, 8), 4)), dim3(256), 0, st, rows, (int)N, stride,
                       tab_coarse.as<unsigned long long>(), lc_coarse, km->out_side.map.as<int>(), ctl);
    SPC_LAUNCH_CHECK();
    SPC_TRY(masks_from_map<27>(km->out_side.map.as<int>(), U, km->out_side.mask.as<unsigned>(), ctl, st));
  } else if (!transposed) {
    km->n_in = N;
    km->n_out = needs_coarse ? U : N;
    const int4* qrows = needs_coarse ? coarse_rows.as<int4>() : rows;
    SPC_TRY(alloc_side(km->out_side, km->n_out, V, st));
    int* mp = km->out_side.map.as<int>();
    unsigned* mk = km->out_side.mask.as<unsigned>();
    const unsigned long long* tf = fine;
    // (a dilated map probes like any other stride-1 map, from its derived output points)
    status = K == 3   ? launch_probe<3>(false, qrows, km->n_out, stride, tf, lc_fine, mp, mk, ctl, st)
             : K == 2 ? launch_probe<2>(false, qrows, km->n_out, stride, tf, lc_fine, mp, mk, ctl, st)
                      : launch_probe<1>(false, qrows, km->n_out, stride, tf, lc_fine, mp, mk, ctl, st);
    SPC_TRY(status);
  } else {
    km->n_in = needs_coarse ? U : N;
    km->n_out = N;
    const unsigned long long* tab = needs_coarse ? tab_coarse.as<unsigned long long>() : fine;
    SPC_TRY(alloc_side(km->out_side, km->n_out, V, st));
    int* mp = km->out_side.map.as<int>();
    unsigned* mk = km->out_side.mask.as<unsigned>();
    const int lc = needs_coarse ? lc_coarse : lc_fine;
    status = K == 3   ? launch_probe<3>(true, rows, N, stride, tab, lc, mp, mk, ctl, st)
             : K == 2 ? launch_probe<2>(true, rows, N, stride, tab, lc, mp, mk, ctl, st)
                      : launch_probe<1>(true, rows, N, stride, tab, lc, mp, mk, ctl, st);
    SPC_TRY(status);
  }
  km->out_side.ready = true;

  if (!needs_coarse || from_inputs) {  // (from_inputs: duplicate rows only show up in the scatter)
    SPC_TRY(read_ctl(ctl, &h, st));
    // (the probe ran before this synchronisation: its pair count is final)
    if (from_inputs && h.entries != h.pairs) h.flags |= FLAG_DUP;  // two rows wrote one entry
    if (h.flags & FLAG_SORT) return kRetryGeneralSort;
    km->build_status = flags_status(h.flags);
    if (!(async && K == 3 && km->submanifold())) SPC_TRY(km->build_status);  // (an unwaited build's verdict is spconv_kmap_status's)
    km->n_pairs = (int64_t)h.pairs;
  }

  // coordinate sets kept for the export calls and for the next layer of a network
  if (!transposed) {
    if (needs_coarse) {
      std::swap(km->in_coords.p, own_rows.p);
      std::swap(km->in_coords.bytes, own_rows.bytes);
      std::swap(km->out_coords.p, coarse_rows.p);
      std::swap(km->out_coords.bytes, coarse_rows.bytes);
    } else {
      std::swap(km->in_coords.p, own_rows.p);
      std::swap(km->in_coords.bytes, own_rows.bytes);  // P_out == P_in: out_coords stays empty
    }
  } else {
    std::swap(km->out_coords.p, own_rows.p);
    std::swap(km->out_coords.bytes, own_rows.bytes);
    if (needs_coarse) {
      std::swap(km->in_coords.p, coarse_rows.p);
      std::swap(km->in_coords.bytes, coarse_rows.bytes);
    }  // stride 1: P_in == the caller's rows: in_coords stays empty
  }
  // temporaries (tables, key lists) go back to the pool here; the stream has either been
  // synchronised (stride 1) or later work on it is ordered after the kernels that read them
  *out = km.release();
  return SPCONV_OK;
}
}  // namespace

int kmap_build_in_side(spconv_kmap* km, hipStream_t st) {
  if (km->in_side.ready) return SPCONV_OK;
  const int V = km->V;
  if (km->in_side.cands.p) {
    SideMap& side = km->in_side;
    side.rows = km->n_in;
    side.rows_pad = round_up(side.rows, kRowPad);
    SPC_TRY(side.map.alloc((size_t)side.rows_pad * V * sizeof(int)));
    SPC_TRY(side.mask.alloc((size_t)side.rows_pad * sizeof(unsigned)));
    const dim3 grid((unsigned)(side.rows_pad / 64));
    const int4* const rows = km->in_coords.as<int4>();
    if (V == 27)
      hipLaunchKernelGGL(k_in_side<3>, grid, dim3(256), 0, st, rows, km->in_side.cands.as<int>(), (long long)side.rows, side.map.as<uint4>(),
                         side.mask.as<unsigned>());
    else
      hipLaunchKernelGGL(k_in_side<2>, grid, dim3(256), 0, st, rows, km->in_side.cands.as<int>(), (long long)side.rows, side.map.as<uint4>(),
                         side.mask.as<unsigned>());
    SPC_LAUNCH_CHECK();
    side.ready = true;
    // Nothing else reads them: the build that wrote them was waited for, so their next user on this stream comes behind the launch above.
    // (Under capture that launch runs at the replays.)
    if (!capturing(st)) side.cands.release();
    return SPCONV_OK;
  }
  SPC_TRY(alloc_side(km->in_side, km->n_in, V, st, true));
  if (km->n_in > 0) {
    const long long entries = (long long)km->n_out * V;
    if (entries > 0) {
      hipLaunchKernelGGL(k_scatter_in_side, dim3(blocks_for(entries, 256)), dim3(256), 0, st,
                         km->out_side.map.as<int>(), entries, V, km->in_side.map.as<int>());
      SPC_LAUNCH_CHECK();
    }
    const int* tm = km->in_side.map.as<int>();
    unsigned* tk = km->in_side.mask.as<unsigned>();
    SPC_TRY(V == 27  ? masks_from_map<27>(tm, km->n_in, tk, nullptr, st)
            : V == 8 ? masks_from_map<8>(tm, km->n_in, tk, nullptr, st)
                     : masks_from_map<1>(tm, km->n_in, tk, nullptr, st));
  }
  km->in_side.ready = true;
  return SPCONV_OK;
}

// The kmap of the transposed convolution that pairs with src: the same pairs with inputs and
// outputs exchanged.  Its output-stationary table is src's input-side table and the other way
// round, so no table is built and nothing is probed: one scatter pass (unless src has its input
// side already) and device-to-device copies.
int kmap_pointwise(spconv_kmap* src, int on_outputs, hipStream_t st, spconv_kmap** out) {
  if (src->pending) SPC_TRY(kmap_status(src, st));  // a failed build has no rows to stand on
  std::unique_ptr<spconv_kmap> km(new (std::nothrow) spconv_kmap);
  if (!km) return SPCONV_ENOMEM;
  const int64_t rows = on_outputs ? src->n_out : src->n_in;
  km->K = 1;
  km->V = 1;
  km->stride = 1;
  km->transposed = 0;
  km->n_in = km->n_out = km->n_pairs = rows;
  km->build_stream = st;
  km->last_stream = st;
  SideMap& side = km->out_side;
  side.rows = rows;
  side.rows_pad = round_up(rows > 0 ? rows : 1, kRowPad);
  SPC_TRY(side.map.alloc((size_t)side.rows_pad * sizeof(int)));
  SPC_TRY(side.mask.alloc((size_t)side.rows_pad * sizeof(unsigned)));
  hipLaunchKernelGGL(k_identity_map, dim3(blocks_for(side.rows_pad, 256)), dim3(256), 0, st, side.map.as<int>(),
                     side.mask.as<unsigned>(), (long long)rows, (long long)side.rows_pad);
  SPC_LAUNCH_CHECK();
  side.ready = true;
  // Which buffer of src holds that side's rows: a kmap keeps the caller's rows and, for stride > 1,
  // the coarse set; with stride 1 the two sets are one (in_coords of a forward kmap, out_coords of
  // a transposed one).
  const DevBuf* from;
  if (!src->transposed)
    from = (on_outputs && (src->stride > 1 || src->dilated)) ? &src->out_coords : &src->in_coords;
  else
    from = (!on_outputs && src->stride > 1) ? &src->in_coords : &src->out_coords;
  if (rows == 0 || !from->p) {
    SPC_TRY(km->in_coords.alloc(16));
  } else {
    SPC_TRY(km->in_coords.alloc((size_t)rows * 16));
    SPC_HIP(hipMemcpyAsync(km->in_coords.p, from->p, (size_t)rows * 16, hipMemcpyDeviceToDevice, st));
  }
  *out = km.release();
  return SPCONV_OK;
}

int kmap_transpose(spconv_kmap* src, hipStream_t st, spconv_kmap** out) {
  if (src->dilated) return SPCONV_EINVAL;  // (no build call returns the transposed partner of a dilated map)
  if (src->pending) SPC_TRY(kmap_status(src, st));  // a failed build has no transpose
  SPC_TRY(kmap_build_in_side(src, st));
  // The transposed convolution's output-stationary table is the source's input-side table and the
  // other way round, and its coordinate sets are the source's with the roles exchanged: the two
  // kmaps share all four buffers (and whatever plans get cached on the tables); nothing is copied.
  // A kmap keeps the caller's rows and, for stride > 1, the coarse set; with stride 1 the two sets
  // are one and only the caller's rows are kept (in_coords of a forward kmap, out_coords of a
  // transposed one), the other buffer stays empty.
  auto none = []() { return std::make_shared<DevBuf>(); };
  std::shared_ptr<DevBuf> in_rows, out_rows;
  if (!src->transposed) {
    out_rows = src->in_coords_ref;
    in_rows = src->stride > 1 ? src->out_coords_ref : none();
  } else {
    in_rows = src->out_coords_ref;
    out_rows = src->stride > 1 ? src->in_coords_ref : none();
  }
  std::unique_ptr<spconv_kmap> km(new (std::nothrow) spconv_kmap(src->in_ref, src->out_ref, in_rows, out_rows));
  if (!km) return SPCONV_ENOMEM;
  km->K = src->K;
  km->V = src->V;
  km->stride = src->stride;
  km->transposed = src->transposed ? 0 : 1;
  km->n_in = src->n_out;
  km->n_out = src->n_in;
  km->n_pairs = src->n_pairs;
  km->build_stream = st;
  km->last_stream = st;
  *out = km.release();
  return SPCONV_OK;
}

int kmap_count_pairs(spconv_kmap* km, hipStream_t st, int64_t* per_k) {
  if (km->pending && !per_k) return kmap_status(km, st) == SPCONV_EHIP ? SPCONV_EHIP : SPCONV_OK;
  unsigned long long h[32] = {0};
  if (km->n_out > 0) {
    DevBuf counts;
    SPC_TRY(counts.alloc(32 * sizeof(unsigned long long)));
    SPC_TRY(fill_u32(counts.p, 64, 0u, st));
    const unsigned blocks = (unsigned)std::min<int64_t>(ceil_div(km->n_out, 256), 1024);
    hipLaunchKernelGGL(k_count_pairs, dim3(blocks), dim3(256), 0, st, km->out_side.mask.as<unsigned>(),
                       (int)km->n_out, counts.as<unsigned long long>());
    SPC_LAUNCH_CHECK();
    SPC_HIP(hipMemcpyAsync(h, counts.p, sizeof(h), hipMemcpyDeviceToHost, st));
    SPC_HIP(hipStreamSynchronize(st));
  }
  int64_t total = 0;
  for (int k = 0; k < km->V; ++k) {
    total += (int64_t)h[k];
    if (per_k) per_k[k] = (int64_t)h[k];
  }
  km->n_pairs = total;
  return SPCONV_OK;
}

namespace {
// The 125-bit mask of a K = 5 row from its planes' 25-bit masks: bit k of the row's mask is bit
// k % 32 of word k / 32, and k = 25 g + j.
__global__ void __launch_bounds__(256) k_join_masks5(Planes5 pl, long long rows, uint4* __restrict__ dst) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  unsigned long long lo = 0, hi = 0;  // bits 0..63, 64..127
#pragma unroll
  for (int g = 0; g < 5; ++g) {
    const unsigned long long m = pl.mask[g][r];
    const int at = 25 * g;
    if (at < 64) {
      lo |= m << at;
      if (at + 25 > 64) hi |= m >> (64 - at);
    } else {
      hi |= m << (at - 64);
    }
  }
  dst[r] = make_uint4((unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32));
}
}  // namespace

int kmap_export_mask_words(const spconv_kmap* km, uint32_t* dst, hipStream_t st) {
  if (km->groups.size() != 5) return SPCONV_EINVAL;
  Planes5 pl{};
  for (int g = 0; g < 5; ++g) pl.mask[g] = km->groups[(size_t)g]->out_side.mask.as<unsigned>();
  hipLaunchKernelGGL(k_join_masks5, dim3(blocks_for(km->n_out, 256)), dim3(256), 0, st, pl, (long long)km->n_out,
                     reinterpret_cast<uint4*>(dst));
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

}  // namespace spc

spconv_kmap::~spconv_kmap() {
  if (pending_host) {  // the copy into the pinned block must have landed before the block is reused
    spc::HostCtlHandle::finish(pending_host);
  }
}
