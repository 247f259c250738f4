// The library's own row order, for calls that leave the configuration to it: rows with equal or similar
// neighbour masks next to each other (the bitmask sorting of Section 2.2.3), made in three short launches.
//
// A full sort by the 27-bit mask takes three digit passes over all rows (100k rows: 12.6 + 11.8 + 11.0 us and 8.6 us for
// the reordered map).  What the kernels need is less: blocks of 16 and tiles of 64 to 256 rows whose masks overlap.
// So the rows go into 256 buckets first (any corner neighbour; the edge neighbours in six pairs; faces along z), one stable
// counting pass whose counter matrix is small enough to be summed by every workgroup, and then
// each stretch of 2048 places is sorted in LDS by 20 bits of the mask.  Which bits matter most: the offsets that few
// rows have (corners 4 %, edges 20 %, faces 40 % of the rows of a LiDAR-like scan) come first, so that the rows that
// have one stand together instead of one in every block.  Executed / valid pairs of blocks of 16 rows, tiles of 64,
// of 128 (100k-voxel scan; 300k-voxel room): this order 1.28, 1.55, 1.71; 1.04, 1.12, 1.21; the full sort by the plain
// mask 1.22, 1.50, 1.74; 1.02, 1.04, 1.06; map order 4.37, 5.64, 5.85; 2.44, 2.76, 2.78.
#include "common.h"
#include "lds_tiles.h"

#include <algorithm>

namespace spc {
namespace {

constexpr int kBucketBits = 8, kBuckets = 1 << kBucketBits;
constexpr int kCountThreads = 256;
constexpr int kScatterThreads = 1024, kScatterWaves = 16;
constexpr int kMaxCountWgs = 256;               // rows of the counter matrix
constexpr int kChunk = 2048;                    // places that are sorted together in LDS
constexpr int kPlaceBits = 11;
constexpr int kLocalThreads = 1024, kLocalWaves = 16, kLocalItems = kChunk / kLocalThreads;
constexpr int kKeyBits = 20, kDigitBits = 7, kDigits = 1 << kDigitBits;
static_assert(kChunk == 1 << kPlaceBits && kBuckets == kCountThreads && kLocalItems == 2 && kScatterThreads == 4 * kBuckets,
              "index arithmetic below");

// V = 27: which corner layers dz = -1, +1 have a neighbour (2 bits), 12 edges, 6 faces.  Other maps: the mask itself.
__device__ __forceinline__ unsigned local_key(unsigned m, int V) {
  if (V != 27) return m & ((1u << kKeyBits) - 1u);
  auto b = [&](int from, int to) { return ((m >> from) & 1u) << to; };
  const unsigned corners = ((m & 0x01040041u) ? 2u : 0u) | ((m & 0x04100104u) ? 1u : 0u);
  const unsigned edges = b(1, 11) | b(7, 10) | b(19, 9) | b(25, 8) | b(3, 7) | b(5, 6) | b(21, 5) | b(23, 4) | b(9, 3) |
                         b(11, 2) | b(15, 1) | b(17, 0);
  const unsigned faces = b(4, 5) | b(10, 4) | b(12, 3) | b(14, 2) | b(16, 1) | b(22, 0);
  return (corners << 18) | (edges << 6) | faces;
}
// V = 27: any corner neighbour, the edge neighbours two by two (two of the four in each coordinate plane: a row of
// a flat surface has the edges of one plane), the face neighbours along z.
__device__ __forceinline__ unsigned bucket_bits(unsigned m, int V) {
  if (V != 27) return V > kBucketBits ? (m >> (V - kBucketBits)) & (kBuckets - 1) : m;
  const unsigned six = m | (m >> 6), two = m | (m >> 2);  // bit i: offsets i and i + 6, i and i + 2
  return (m & 0x05140145u ? 128u : 0u) | ((six >> 1) & 1u) << 6 | ((six >> 19) & 1u) << 5 | ((two >> 3) & 1u) << 4 |
         ((two >> 21) & 1u) << 3 | ((two >> 9) & 1u) << 2 | ((two >> 15) & 1u) << 1 | ((two >> 12) & 1u);
}
// The buckets in the order of their set bits: rows with many neighbours stand at the end of the order, where the
// kernels start (the heaviest tiles first).
struct BucketRanks {
  unsigned short of[kBuckets];
};
constexpr BucketRanks make_bucket_ranks() {
  BucketRanks r{};
  int next = 0;
  for (int bits = 0; bits <= kBucketBits; ++bits)
    for (int b = 0; b < kBuckets; ++b) {
      int n = 0;
      for (int i = 0; i < kBucketBits; ++i) n += (b >> i) & 1;
      if (n == bits) r.of[b] = (unsigned short)next++;
    }
  return r;
}
__device__ const BucketRanks d_ranks = make_bucket_ranks();

// counts[workgroup][bucket] of wg_rows consecutive rows each
__global__ void __launch_bounds__(kCountThreads)
    k_order_count(const unsigned* __restrict__ mask, int rows, int wg_rows, int V, unsigned* __restrict__ counts) {
  __shared__ unsigned cnt[kBuckets];
  for (int d = threadIdx.x; d < kBuckets; d += kCountThreads) cnt[d] = 0;
  __syncthreads();
  const int begin = blockIdx.x * wg_rows, end = min(rows, begin + wg_rows);
  for (int r0 = begin; r0 < end; r0 += 4 * kCountThreads) {
    unsigned at[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + i * kCountThreads + threadIdx.x;
      at[i] = r < end ? d_ranks.of[bucket_bits(mask[r], V)] : kBuckets;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (at[i] < kBuckets) atomicAdd(&cnt[at[i]], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < kBuckets; d += kCountThreads) counts[blockIdx.x * kBuckets + d] = cnt[d];
}

// For every lane: how many lower lanes of the wave hold the same digit, and how many lanes do.
__device__ __forceinline__ void rank_of(unsigned digit, int bits, bool valid, int lane, unsigned* rank, unsigned* peers_out) {
  unsigned long long peers = __ballot(valid);
  for (int b = 0; b < bits; ++b) {
    const bool bit = (digit >> b) & 1u;
    const unsigned long long bal = __ballot(bit);
    peers &= bit ? bal : ~bal;
  }
  *rank = (unsigned)__popcll(peers & ((1ull << lane) - 1ull));
  *peers_out = (unsigned)__popcll(peers);
}

// Rows of one workgroup to their places: bucketed[place] = (local key, row), stable.  The workgroup finds its first
// places by adding up the counter matrix (at most 256 x 256 counters from L2, a quarter of the rows per 256 threads: with 256 threads
// in all, 200k rows took 13 us) instead of waiting for a scan launch.
__global__ void __launch_bounds__(kScatterThreads)
    k_order_scatter(const unsigned* __restrict__ mask, int rows, int wg_rows, int V, const unsigned* __restrict__ counts,
                    uint2* __restrict__ bucketed) {
  __shared__ unsigned off[kScatterWaves][kBuckets];  // of a round of 1024 rows: the waves' counts, then first places
  __shared__ unsigned part_before[4][kBuckets], part_all[4][kBuckets], wave_sum[4], place[kBuckets];
  const int t = threadIdx.x, lane = t & 63, wib = t >> 6, d = t & (kBuckets - 1), part = t / kBuckets;
  const int begin = blockIdx.x * wg_rows, end = min(rows, begin + wg_rows);
  unsigned m = begin + t < end ? mask[begin + t] : 0u;
  {
    unsigned before = 0, all = 0;
    constexpr int R = 16;  // rows in flight: a load that waits for the one before it costs a round trip each
    for (int w0 = part; w0 < (int)gridDim.x; w0 += 4 * R) {
      unsigned c[R];
#pragma unroll
      for (int i = 0; i < R; ++i) c[i] = w0 + 4 * i < (int)gridDim.x ? counts[(w0 + 4 * i) * kBuckets + d] : 0u;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        all += c[i];
        before += w0 + 4 * i < (int)blockIdx.x ? c[i] : 0u;
      }
    }
    part_before[part][d] = before;
    part_all[part][d] = all;
  }
  __syncthreads();
  unsigned incl = 0, all = 0;
  if (t < kBuckets) {
    for (int i = 0; i < 4; ++i) all += part_all[i][t];
    incl = all;
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    if (lane == 63) wave_sum[wib] = incl;
  }
  __syncthreads();
  if (t < kBuckets) {
    unsigned at = incl - all;
    for (int i = 0; i < 4; ++i) at += part_before[i][t];
    for (int w = 0; w < wib; ++w) at += wave_sum[w];
    place[t] = at;  // next place of the bucket
  }
  for (int r0 = begin; r0 < end; r0 += kScatterThreads) {
    const int r = r0 + t;
    const bool valid = r < end;
    if (r0 > begin) m = valid ? mask[r] : 0u;
    for (int i = t; i < kScatterWaves * kBuckets; i += kScatterThreads) (&off[0][0])[i] = 0;
    __syncthreads();
    const unsigned bkt = d_ranks.of[bucket_bits(m, V)];
    unsigned rank, peers;
    rank_of(bkt, kBucketBits, valid, lane, &rank, &peers);
    if (valid && rank == 0) off[wib][bkt] = peers;
    __syncthreads();
    if (t < kBuckets) {
      unsigned at = place[t], c[kScatterWaves];  // (read before the first is written: else each read waits for the write before it)
#pragma unroll
      for (int w = 0; w < kScatterWaves; ++w) c[w] = off[w][t];
#pragma unroll
      for (int w = 0; w < kScatterWaves; ++w) {
        off[w][t] = at;
        at += c[w];
      }
      place[t] = at;
    }
    __syncthreads();
    const unsigned at = off[wib][bkt] + rank;
    if (valid && at < (unsigned)rows) bucketed[at] = make_uint2(local_key(m, V), (unsigned)r);
    __syncthreads();
  }
}

// Sorts a stretch of 2048 places by the local key (stable: three digits in LDS), and writes what a plan consists
// of: the rows' order, the reordered map and the masks of its 16-row blocks.  Where there are fewer stretches than CUs,
// gridDim.y workgroups sort the same one and each writes its share (the reordering is most of the work).
__global__ void __launch_bounds__(kLocalThreads)
    k_order_local(const uint2* __restrict__ bucketed, const unsigned* __restrict__ mask, const int* __restrict__ map, int V,
                  int rows, long long rows_pad, long long n_blocks, int* __restrict__ perm, int* __restrict__ reordered,
                  unsigned* __restrict__ blkmask) {
  __shared__ int row_of[kChunk];            // by place within the bucket order
  __shared__ unsigned comp[kChunk];         // key << 11 | place
  __shared__ __align__(8) unsigned off[kLocalWaves][kDigits];
  __shared__ int src_of[kChunk];            // rows in the final order
  const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
  const long long base = (long long)blockIdx.x * kChunk;
  unsigned v[kLocalItems];
#pragma unroll
  for (int i = 0; i < kLocalItems; ++i) {
    const int at = wib * (64 * kLocalItems) + i * 64 + lane;
    const uint2 e = base + at < rows ? bucketed[base + at] : make_uint2((1u << kKeyBits) - 1u, 0xFFFFFFFFu);  // padding last
    row_of[at] = (int)e.y;
    v[i] = (e.x << kPlaceBits) | (unsigned)at;
  }
  for (int shift = kPlaceBits; shift < kPlaceBits + kKeyBits; shift += kDigitBits) {
    const int bits = min(kDigitBits, kPlaceBits + kKeyBits - shift);
    for (int d = threadIdx.x; d < kLocalWaves * kDigits; d += kLocalThreads) (&off[0][0])[d] = 0;
    __syncthreads();
    unsigned digit[kLocalItems], rank[kLocalItems];
#pragma unroll
    for (int i = 0; i < kLocalItems; ++i) {
      digit[i] = (v[i] >> shift) & ((1u << bits) - 1u);
      unsigned peers;
      rank_of(digit[i], bits, true, lane, &rank[i], &peers);
      const unsigned have = off[wib][digit[i]];
      __builtin_amdgcn_wave_barrier();
      if (rank[i] == 0) off[wib][digit[i]] = have + peers;
      __builtin_amdgcn_wave_barrier();
      rank[i] += have;
    }
    __syncthreads();
    if (threadIdx.x < 64) {  // first places: digits in order, within a digit the waves in order; two digits per lane
      unsigned c[2][kLocalWaves], both = 0;  // (read before the first is written: else each read waits for the write before it)
#pragma unroll
      for (int w = 0; w < kLocalWaves; ++w) {
        const uint2 v = *reinterpret_cast<const uint2*>(&off[w][2 * lane]);
        c[0][w] = v.x, c[1][w] = v.y;
        both += v.x + v.y;
      }
      unsigned incl = both;
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
      }
      unsigned run = incl - both;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int w = 0; w < kLocalWaves; ++w) {
          const unsigned n = c[d][w];
          c[d][w] = run;
          run += n;
        }
#pragma unroll
      for (int w = 0; w < kLocalWaves; ++w) *reinterpret_cast<uint2*>(&off[w][2 * lane]) = make_uint2(c[0][w], c[1][w]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kLocalItems; ++i) comp[off[wib][digit[i]] + rank[i]] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kLocalItems; ++i) v[i] = comp[wib * (64 * kLocalItems) + i * 64 + lane];
  }
  const int share = kChunk / gridDim.y, lo = blockIdx.y * share;  // (a power of two, at least 128)
  unsigned m[kLocalItems];
#pragma unroll
  for (int i = 0; i < kLocalItems; ++i) {
    const int at = wib * (64 * kLocalItems) + i * 64 + lane;
    const int src = row_of[v[i] & (kChunk - 1)];
    src_of[at] = src;
    const bool mine = at >= lo && at < lo + share;
    if (mine && base + at < rows_pad) perm[base + at] = src;
    m[i] = mine && src >= 0 ? mask[src] : 0u;
  }
  sync_lds();  // (the masks are still on their way while the map's rows are asked for)
  // e / V by a multiply: (e + 0.5) / V stays 0.5 / 27 away from every integer for e < 55296
  const long long first = base + lo;
  const int n = first >= rows_pad ? 0 : (int)min((long long)share, rows_pad - first) * V;
  int* dst = reordered + first * V;
  const float inv = 1.0f / (float)V;
  constexpr int U = 14;  // loads in flight per thread
  for (int e0 = threadIdx.x; e0 < n; e0 += U * kLocalThreads) {
    int val[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kLocalThreads;
      val[u] = -1;
      if (e < n) {
        const int rr = (int)(((float)e + 0.5f) * inv), sr = src_of[lo + rr];
        if (sr >= 0) val[u] = map[(long long)sr * V + (e - rr * V)];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (e0 + u * kLocalThreads < n) dst[e0 + u * kLocalThreads] = val[u];
  }
#pragma unroll
  for (int i = 0; i < kLocalItems; ++i) {
    const int at = wib * (64 * kLocalItems) + i * 64 + lane;
    for (int o = 1; o < 16; o <<= 1) m[i] |= __shfl_xor(m[i], o);
    const long long block = (base + at) / 16;
    if (at >= lo && at < lo + share && (lane & 15) == 0 && block < n_blocks) blkmask[block] = m[i];
  }
}

}  // namespace

int order_rows(const SideMap& side, int V, IgemmPlan& p, hipStream_t st) {
  const int rows = (int)p.rows;
  int wg_rows = 1024;
  while (ceil_div(rows, wg_rows) > kMaxCountWgs) wg_rows *= 2;
  const unsigned wgs = (unsigned)ceil_div(rows, wg_rows);
  DevBuf tmp;  // (returns to the pool while the stream may still use it; later users are ordered behind)
  const size_t bucketed_bytes = (size_t)rows * sizeof(uint2);
  SPC_TRY(tmp.alloc(bucketed_bytes + (size_t)wgs * kBuckets * sizeof(unsigned)));
  uint2* bucketed = tmp.as<uint2>();
  unsigned* counts = reinterpret_cast<unsigned*>(tmp.as<char>() + bucketed_bytes);
  const unsigned* mask = side.mask.as<unsigned>();
  hipLaunchKernelGGL(k_order_count, dim3(wgs), dim3(kCountThreads), 0, st, mask, rows, wg_rows, V, counts);
  SPC_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_order_scatter, dim3(wgs), dim3(kScatterThreads), 0, st, mask, rows, wg_rows, V, counts, bucketed);
  SPC_LAUNCH_CHECK();
  const unsigned chunks = (unsigned)ceil_div(p.rows_pad, kChunk);
  unsigned shares = 16;  // (9k rows with 4: 12.5 us, so 10.5; two workgroups on one CU take longer than one after the other: 200k rows 27, 19.6)
  while (shares > 1 && chunks * shares > 256) shares /= 2;
  hipLaunchKernelGGL(k_order_local, dim3(chunks, shares), dim3(kLocalThreads), 0, st, bucketed, mask,
                     side.map.as<int>(), V, rows, (long long)p.rows_pad, (long long)p.n_tiles, p.perm.as<int>(), p.maps.as<int>(),
                     p.tilemask.as<unsigned>());
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

}  // namespace spc
