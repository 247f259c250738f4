// Weight-gradient kernels (Sections 4.2, 6.2): dW[k] = sum over present pairs
// (n, j = M[n][k]) of x[j]^T . dy[n].
//
// The reduction runs over output rows, the long inner loop the paper singles
// out.  Here it walks the compacted pair list of one offset (the
// weight-stationary view of the map, Section 2.2.1), so no multiply is spent
// on absent neighbours and the row order of the map does not matter.
//
// Work split.  Each offset's pairs are cut into pieces of nearly equal length, one per workgroup.  A piece leaves an fp32
// partial tile; a second kernel adds the tiles of each offset in order, so results are bit-reproducible.  The number
// of pieces weighs the time that a piece takes against the tiles that are written and read back, and goes down to whole
// rounds of one workgroup per CU (split_length); at most as many run as the GPU holds at once, unless a layer's tiles alone
// fill it (split_for).
//
// What bounds it is the gather: every pair's two rows cross the cache hierarchy once per column or row of tiles,
// so the tile is as wide as the layer up to 256 x 256 (pick_tile).  Rows go straight into LDS (batches of 32 pairs, two to three of them
// in flight ahead of the one that is multiplied, each load waited for by count); the matrix instructions need the
// pair index contiguous per lane, which the transposing LDS read (ds_read_b64_tr_b16) delivers.  Fragments of
// the next batch are read while the matrix cores work on this one.  Narrow layers (one wave's tile) give every
// wave batches of its own: no barrier, and the waves' sums meet in LDS at the end of the piece.
//
// Measured, both kernels of a call (before: 128 x 128 tiles staged through registers, fp32 without matrix cores): 2.9M
// pairs bf16, 256 -> 256: 793 -> 434 us, 2.95 GB gathered at 6.8 TB/s (random rows of 128-byte lines come from the
// last-level cache at about 7 TB/s); 96 -> 96: 218 -> 191 us (192-byte rows touch two lines); 32 -> 32: 98 -> 86 us (64-byte
// rows: 5 TB/s at best).  680k pairs f16, 64 -> 128: 57 -> 48 us.  128k pairs fp32, 64 -> 64: 112 -> 26 us.
#include "common.h"
#include "lds_tiles.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>
#include <utility>

namespace spc {
namespace {

struct Split {
  int pieces;    // at most so many (grid, partial tiles)
  int length;    // pairs of a piece as asked for, or 0: chosen by
  float weight;  // sqrt(time of a pair in a piece / time of a partial tile), and at least
  int unit;      // so many
  int per_round;  // pieces that make one workgroup per CU
};

struct WgradParams {
  const void* feats;   // [n_in][C_in]
  const void* dout;    // [n_out][C_out]
  const int2* pairs;   // (n, j), offset-major
  const int* seg;      // [V+1]
  float* partial;      // [piece][C_in][C_out]
  unsigned feats_bytes, dout_bytes, pairs_bytes;
  int C_in, C_out, V;
  Split split;
};

constexpr unsigned kNoRow = 0xFFFFC000u;  // beyond every buffer

// Pairs per piece; computed by every workgroup, as the pair count may only be known on the device.
// g pieces take time ~ pairs / g (a workgroup's serial part) + g * (a tile written and read): least at g ~ sqrt(pairs).
// Long pieces then go down to whole rounds of one workgroup per CU, each offset's last piece counted: two workgroups of a CU
// gather at half the rate each, and the launch waits for the CUs that have one more (421k pairs 128 -> 128, 410 pieces 47.2 us,
// 249 pieces 40.9; 256 -> 128, 604 workgroups 80.0, 510 69.1).  Not where that takes too many of them (271k pairs 256 ->
// 128, 496 workgroups 47.9 us, 256 57.1), nor where pieces are short, so that their start is what counts (127k pairs 256
// -> 128: 32.9 us, in one round 35.3).
__device__ __forceinline__ int split_length(const Split& s, int pairs, int V) {
  if (s.length > 0) return s.length;
  int g = min(s.pieces - V, (int)(s.weight * sqrtf((float)pairs)) + 1);
  const int whole = (g + V) / s.per_round * s.per_round - V;
  const int least = s.per_round == 256 ? g / 2 : g - g / 4;  // (a single column of tiles: rounds are finer)
  if (whole >= least && pairs / g >= 900) g = whole;
  return max(s.unit, (pairs + g - 1) / g);
}
// Lane k < V of a wave: the pieces of the offsets before k, and of k.
struct Pieces {
  int before, count;
};
__device__ __forceinline__ Pieces pieces_of(const Split& s, int bound, int V, int lane) {  // bound: lane k <= V holds seg[k]
  const int length = split_length(s, __builtin_amdgcn_readlane(bound, V), V);
  const int pairs = __shfl_down(bound, 1) - bound;
  const int count = lane < V ? (pairs + length - 1) / length : 0;
  int incl = count;
  for (int o = 1; o < 32; o <<= 1) {
    const int up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  return {incl - count, count};
}

template <int N> __device__ __forceinline__ void wait_loads() {  // all but the N youngest; own LDS reads are done as well
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"i"(N) : "memory");
}

// TI x TO (channels of x, of dy) per workgroup; NWI x NWO waves share a batch, or (NWK > 1) each wave has its own.
// S stages.
template <typename T, int TI, int TO, int NWI, int NWO, int NWK, int S> struct WgradShape {
  static constexpr int E = (int)sizeof(T), CE = 16 / E;  // bytes and chunk length of an element
  static constexpr int BP = E == 2 ? 32 : 16;            // pairs of a batch
  static constexpr int NW = NWI * NWO;
  static constexpr int WI = TI / NWI, WO = TO / NWO, IB = WI / 16, OB = WO / 16;
  static constexpr int x_bytes = BP * TI * E, d_bytes = BP * TO * E, stage = x_bytes + d_bytes;
  static constexpr int LX = x_bytes / 1024, LD = d_bytes / 1024;  // loads of a stage
  static constexpr int L = (LX + LD) / NW;                        // per wave
  static constexpr int idx_bytes = BP * 8;
  static constexpr int R = 2 * S;                        // index ring
  static constexpr int group = S * stage + R * idx_bytes;  // LDS of a wave group
  static constexpr int sums = NWK > 1 ? TI * TO * 4 : 0;
  static constexpr int total = NWK * (group > sums ? group : sums);
  static constexpr int threads = NW * NWK * 64;
  static_assert(NW == 1 || NWK == 1, "");
  static_assert((LX + LD) % NW == 0 && x_bytes % 1024 == 0 && d_bytes % 1024 == 0, "whole loads");
  static_assert(L * (S - 2) + S - 2 < 64, "vmcnt");
};

// Where chunk c (16 bytes) of row r of a staged batch stands.  16-bit types: the transposing read of 32 lanes takes rows
// r..r+3 and r+8..r+11 at one 32-byte block each; fp32: four rows at one 64-byte block.  Eight (four) blocks span
// the LDS banks, so the block number is XORed (six blocks: rotated) by the row.
template <int E, int CPR> __device__ __forceinline__ int chunk_block_shift(int r) {
  if constexpr (E == 4) return CPR >= 16 ? (r & 3) : (r >> 1) & 1;
  else if constexpr (CPR == 4) return (r >> 3) & 1;
  else if constexpr (CPR == 8) return ((r >> 1) & 1) | (((r >> 3) & 1) << 1);
  else if constexpr (CPR == 12) return (r >> 3) & 1;
  else return (r & 3) | (((r >> 3) & 1) << 2);
}
// block b of row r stands at block place_of(b), and place q holds block block_at(q)
template <int E, int CPR> __device__ __forceinline__ int place_of(int b, int r) {
  if constexpr (E == 2 && CPR == 12) {
    const int q = b + chunk_block_shift<E, CPR>(r);
    return q >= 6 ? q - 6 : q;
  } else {
    return b ^ chunk_block_shift<E, CPR>(r);
  }
}
template <int E, int CPR> __device__ __forceinline__ int block_at(int q, int r) {
  if constexpr (E == 2 && CPR == 12) {
    const int b = q - chunk_block_shift<E, CPR>(r);
    return b < 0 ? b + 6 : b;
  } else {
    return q ^ chunk_block_shift<E, CPR>(r);
  }
}

template <typename T, int TI, int TO, int NWI, int NWO, int NWK, int S>
__global__ void __launch_bounds__(NWI* NWO* NWK * 64) k_wgrad(const WgradParams p) {
  typedef WgradShape<T, TI, TO, NWI, NWO, NWK, S> W;
  constexpr int E = W::E, CE = W::CE, BP = W::BP, NW = W::NW, IB = W::IB, OB = W::OB, L = W::L, R = W::R;
  constexpr int CX = TI / CE, CD = TO / CE;     // chunks of a staged row
  constexpr int BC = E == 2 ? 2 : 4;            // chunks of a block (16 channels)
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = NWK > 1 ? wave_all : 0, wave = NWK > 1 ? 0 : wave_all;
  const int wi = wave / NWO, wo = wave % NWO;
  const int fa = lane & 15, fg = lane >> 4;
  const int ci0 = blockIdx.y * TI, co0 = blockIdx.z * TO;
  unsigned char* const my = smem + grp * W::group;   // stages, then the index ring
  const unsigned lds = (unsigned)(size_t)(__attribute__((address_space(3))) void*)my;
  constexpr int kIdx = S * W::stage;

  const int bound = lane <= p.V ? p.seg[lane] : 0x7FFFFFFF;  // lane k: where offset k's pairs begin
  int k, begin, end;
  {
    const Pieces pc = pieces_of(p.split, bound, p.V, lane);
    k = __popcll(__ballot(lane < p.V && pc.before + pc.count <= (int)blockIdx.x));
    if (k >= p.V) return;
    const int q = (int)blockIdx.x - __builtin_amdgcn_readlane(pc.before, k);
    const int first = __builtin_amdgcn_readlane(bound, k), all = __builtin_amdgcn_readlane(bound, k + 1) - first;
    const int count = __builtin_amdgcn_readlane(pc.count, k), length = (all + count - 1) / count;
    begin = first + q * length;
    end = max(begin, min(first + all, begin + length));  // (may be empty: the tile is then zero)
  }

  const u32x4 x_rsrc = rsrc_of(p.feats, p.feats_bytes), d_rsrc = rsrc_of(p.dout, p.dout_bytes);
  const u32x4 p_rsrc = rsrc_of(p.pairs, p.pairs_bytes);
  const unsigned x_row = (unsigned)p.C_in * E, d_row = (unsigned)p.C_out * E;

  // this wave's loads of a stage: lane -> row of the batch, byte offset within the row (kNoRow: no such channel)
  int l_row[L];
  unsigned l_off[L];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int j = wave * L + i;
    if (j < W::LX) {
      const int q = j * 64 + lane, r = q / CX, c = q % CX;
      const int ch = (block_at<E, CX>(c / BC, r) * BC + c % BC) * CE + ci0;
      l_row[i] = r;
      l_off[i] = ch < p.C_in ? (unsigned)ch * E : kNoRow;
    } else {
      const int q = (j - W::LX) * 64 + lane, r = q / CD, c = q % CD;
      const int ch = (block_at<E, CD>(c / BC, r) * BC + c % BC) * CE + co0;
      l_row[i] = r;
      l_off[i] = ch < p.C_out ? (unsigned)ch * E : kNoRow;
    }
  }
  // fragment addresses within a stage
  unsigned xa[IB], da[OB];
  {
    const int r = E == 2 ? 8 * fg + (fa >> 2) : fg;
    const int in = E == 2 ? (fa & 3) * 8 : fa * 4;
#pragma unroll
    for (int i = 0; i < IB; ++i) xa[i] = (unsigned)(r * TI * E + place_of<E, CX>(wi * IB + i, r) * BC * 16 + in);
#pragma unroll
    for (int i = 0; i < OB; ++i) da[i] = (unsigned)(W::x_bytes + r * TO * E + place_of<E, CD>(wo * OB + i, r) * BC * 16 + in);
  }
  auto frag = [&](const unsigned char* at, int pitch) -> u32x4 {
    if constexpr (E == 2) {
      // 16 lanes fetch a 4 x 16 block of [pair][channel] and each receives one column; two reads give the lane's
      // 8 pairs (8 fg .. 8 fg + 7) of its channel
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at + 4 * pitch));
      return __builtin_bit_cast(u32x4, s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    } else {  // pairs fg, 4 + fg, 8 + fg, 12 + fg
      u32x4 v;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = *reinterpret_cast<const unsigned*>(at + t * 4 * pitch);
      return v;
    }
  };

  const int first = begin & ~1;  // (index loads are 16 bytes: two pairs)
  const int batches = max(end - first + BP - 1, 0) / BP;
  const int mine = NWK > 1 ? (batches - grp + NWK - 1) / NWK : batches;  // batches grp, grp + NWK, ...

  auto batch_pair = [&](int b) { return first + (NWK > 1 ? b * NWK + grp : b) * BP; };
  auto load_idx = [&](int b) {  // pair indices of own batch b into the ring; every wave of a group loads the same bytes
    if (lane < BP / 2)
      load_to_lds(p_rsrc, (unsigned)(batch_pair(b) + lane * 2) * 8u, 0, lds + kIdx + (unsigned)(b % R) * W::idx_bytes);
  };
  unsigned src[L];
  auto read_idx = [&](int b) {  // row offsets of own batch b
    const int e0 = batch_pair(b);
    const unsigned char* ring = my + kIdx + (b % R) * W::idx_bytes;
    unsigned row[L];
#pragma unroll
    for (int i = 0; i < L; ++i)
      row[i] = *reinterpret_cast<const unsigned*>(ring + l_row[i] * 8 + ((NW == 1 ? i < W::LX : wave * L + i < W::LX) ? 4 : 0));
#pragma unroll
    for (int i = 0; i < L; ++i) asm volatile("" : "+v"(row[i]));  // (else every read becomes a branch of its own)
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const bool is_x = NW == 1 ? i < W::LX : wave * L + i < W::LX;
      const bool live = (unsigned)(e0 + l_row[i] - begin) < (unsigned)(end - begin);
      const unsigned at = row[i] * (is_x ? x_row : d_row) + l_off[i];
      src[i] = live && l_off[i] != kNoRow ? at : kNoRow;
    }
  };
  auto load_stage = [&](int slot) {
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int j = wave * L + i;
      const bool is_x = NW == 1 ? i < W::LX : j < W::LX;
      load_to_lds(is_x ? x_rsrc : d_rsrc, src[i], 0, lds + slot * W::stage + j * 1024);
    }
  };
  auto sync = [&]() {
    if constexpr (NW > 1) asm volatile("s_barrier" ::: "memory");
  };

  f32x4 acc[OB][IB];
#pragma unroll
  for (int o = 0; o < OB; ++o)
#pragma unroll
    for (int i = 0; i < IB; ++i) acc[o][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  // indices of the first 2 S batches, stages of the first S
#pragma unroll
  for (int b = 0; b < R; ++b) load_idx(b);
  wait_loads<0>();
  sync();
#pragma unroll
  for (int b = 0; b < S; ++b) {
    read_idx(b);
    load_stage(b);
  }
  read_idx(S);
  wait_loads<(S - 1) * L>();
  sync();
  u32x4 x[IB], d[OB];
#pragma unroll
  for (int o = 0; o < OB; ++o) d[o] = frag(my + da[o], TO * E);
#pragma unroll
  for (int i = 0; i < IB; ++i) x[i] = frag(my + xa[i], TI * E);

  int slot = 0;
  for (int b = 0; b < mine; ++b) {
    // batch b + 1 has landed (and the indices of b + S + 1), and everyone holds batch b in registers
    if (b < S - 2) wait_loads<(S - 2) * L>();
    else wait_loads<(S - 2) * (L + 1)>();
    sync();
    load_stage(slot);  // batch b + S
    load_idx(b + 2 * S);
    slot = slot + 1 == S ? 0 : slot + 1;
    read_idx(b + S + 1);
    const unsigned char* next = my + slot * W::stage;
    u32x4 xn[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) xn[i] = frag(next + xa[i], TI * E);
#pragma unroll
    for (int o = 0; o < OB; ++o) {
#pragma unroll
      for (int i = 0; i < IB; ++i) acc[o][i] = mma<T>(d[o], x[i], acc[o][i]);
      d[o] = frag(next + da[o], TO * E);
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) x[i] = xn[i];
  }
  wait_loads<0>();  // (nothing may land in LDS that is used for something else next)

  // a lane holds channels co = 4 fg .. + 3 of row ci = fa of each block
  float* dst = p.partial + (long long)blockIdx.x * p.C_in * p.C_out;
  auto store = [&](int ci, int co, f32x4 v) {
    if (ci < p.C_in && co < p.C_out) *reinterpret_cast<f32x4*>(dst + (long long)ci * p.C_out + co) = v;
  };
  if constexpr (NWK > 1) {
    __syncthreads();
    f32x4* sums = reinterpret_cast<f32x4*>(smem);  // [group][block][lane]
#pragma unroll
    for (int o = 0; o < OB; ++o)
#pragma unroll
      for (int i = 0; i < IB; ++i) sums[(grp * OB * IB + o * IB + i) * 64 + lane] = acc[o][i];
    __syncthreads();
    constexpr int Q = OB * IB / NWK;  // blocks that each group adds up
    static_assert(NWK == 1 || OB * IB % NWK == 0, "");
#pragma unroll
    for (int u = 0; u < Q; ++u) {
      const int blk = grp * Q + u, o = blk / IB, i = blk % IB;
      f32x4 v = sums[blk * 64 + lane];
#pragma unroll
      for (int g = 1; g < NWK; ++g) v += sums[(g * OB * IB + blk) * 64 + lane];
      store(ci0 + i * 16 + fa, co0 + o * 16 + fg * 4, v);
    }
  } else {
#pragma unroll
    for (int o = 0; o < OB; ++o)
#pragma unroll
      for (int i = 0; i < IB; ++i)
        store(ci0 + wi * W::WI + i * 16 + fa, co0 + wo * W::WO + o * 16 + fg * 4, acc[o][i]);
  }
}

// fp32 with more than 32 bits of byte offsets: plain FMA arithmetic, 16 pairs at a time.
__global__ void __launch_bounds__(256) k_wgrad_f32(const WgradParams p) {
  __shared__ float Xs[16][64 + 4];
  __shared__ float Ds[16][64 + 4];
  const int tid = threadIdx.x;
  int begin, end;
  {
    const int lane = tid & 63, bound = lane <= p.V ? p.seg[lane] : 0x7FFFFFFF;
    const Pieces pc = pieces_of(p.split, bound, p.V, lane);
    const int k = __popcll(__ballot(lane < p.V && pc.before + pc.count <= (int)blockIdx.x));
    if (k >= p.V) return;
    const int q = (int)blockIdx.x - __builtin_amdgcn_readlane(pc.before, k);
    const int first = __builtin_amdgcn_readlane(bound, k), all = __builtin_amdgcn_readlane(bound, k + 1) - first;
    const int count = __builtin_amdgcn_readlane(pc.count, k), length = (all + count - 1) / count;
    begin = first + q * length;
    end = max(begin, min(first + all, begin + length));
  }
  const int ci0 = blockIdx.y * 64, co0 = blockIdx.z * 64;
  const float* feats = reinterpret_cast<const float*>(p.feats);
  const float* dout = reinterpret_cast<const float*>(p.dout);
  const int ty = tid / 16, tx = tid % 16;
  const int q = tid / 16, seg4 = (tid % 16) * 4;
  float acc[4][4] = {};
  for (int base = begin; base < end; base += 16) {
    const int e = base + q;
    float4 vx = make_float4(0.f, 0.f, 0.f, 0.f), vd = vx;
    if (e < end) {
      const int2 pr = p.pairs[e];
      if (ci0 + seg4 < p.C_in) vx = *reinterpret_cast<const float4*>(feats + (long long)pr.y * p.C_in + ci0 + seg4);
      if (co0 + seg4 < p.C_out) vd = *reinterpret_cast<const float4*>(dout + (long long)pr.x * p.C_out + co0 + seg4);
    }
    *reinterpret_cast<float4*>(&Xs[q][seg4]) = vx;
    *reinterpret_cast<float4*>(&Ds[q][seg4]) = vd;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = Xs[r][ty * 4 + i];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) b[jj] = Ds[r][tx * 4 + jj];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) acc[i][jj] = fmaf(a[i], b[jj], acc[i][jj]);
    }
    __syncthreads();
  }
  float* dst = p.partial + (long long)blockIdx.x * p.C_in * p.C_out;
  for (int i = 0; i < 4; ++i) {
    const int ci = ci0 + ty * 4 + i;
    if (ci >= p.C_in) continue;
    for (int jj = 0; jj < 4; ++jj) {
      const int co = co0 + tx * 4 + jj;
      if (co < p.C_out) dst[(long long)ci * p.C_out + co] = acc[i][jj];
    }
  }
}

// dW[k][e] = sum of the partial tiles of offset k.  A workgroup covers 64 float4 columns; its four
// waves take the tiles of the offset round-robin (four loads in flight each) and their sums are
// added in wave order, so the order of additions is fixed and results are bit-reproducible.
__global__ void __launch_bounds__(256) k_wgrad_reduce(const float* __restrict__ partial,
                                                      const int* __restrict__ seg, int V, Split split, int elems,
                                                      float* __restrict__ dw) {
  __shared__ float4 part[4][64];
  const int col = threadIdx.x & 63, stripe = threadIdx.x >> 6;
  const int e4 = (blockIdx.x * 64 + col) * 4;
  const int k = blockIdx.y;
  const Pieces pc = pieces_of(split, col <= V ? seg[col] : 0x7FFFFFFF, V, col);
  const int first = __builtin_amdgcn_readlane(pc.before, k), last = first + __builtin_amdgcn_readlane(pc.count, k);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (e4 < elems) {
    int it = first + stripe;
    for (; it + 12 < last; it += 16) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(partial + (long long)(it + 4 * u) * elems + e4);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        s.x += v[u].x;
        s.y += v[u].y;
        s.z += v[u].z;
        s.w += v[u].w;
      }
    }
    for (; it < last; it += 4) {
      const float4 v = *reinterpret_cast<const float4*>(partial + (long long)it * elems + e4);
      s.x += v.x;
      s.y += v.y;
      s.z += v.z;
      s.w += v.w;
    }
  }
  part[stripe][col] = s;
  __syncthreads();
  if (stripe == 0 && e4 < elems) {
    float4 t = part[0][col];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      t.x += part[w][col].x;
      t.y += part[w][col].y;
      t.z += part[w][col].z;
      t.w += part[w][col].w;
    }
    *reinterpret_cast<float4*>(dw + (long long)k * elems + e4) = t;
  }
}

// ---- narrow layers on dense maps: straight from the map ----
// A layer of up to 32 channels on either side has a gradient so small that a wave's registers hold it for J offsets.  Such a wave walks
// batches of 32 map rows, keeps the batch's rows of dy in registers for all of its offsets and gathers their rows of x
// (absent ones are zeros): every row of dy is read once per wave type, V / J times, and in order, not once per pair, and no pair
// list is made (24 us at 300k rows of a room).  300k rows, 2.8M pairs, bf16 32 -> 32: 80 us + list -> 62, 8 -> 32 64 -> 43: the lines
// that 64-byte rows of x lie in, 353 MB, at 6.3 TB/s.  Absent neighbours cost a slot of the address unit and matrix
// instructions, so sparse maps stay with the pairs (100k rows of a LiDAR-like scan, 3.4 pairs a row: 16 us, from the map 23), as
// do 64 channels of dy (300k rows 32 -> 64 95, 102) and maps of fewer pairs than about a million (wgrad_from_map).
// Waves are on their own: batches are dealt to them, a unit (offset of a batch) has J - 1 units in flight behind it, each waited for
// by count; the waves' sums meet in LDS and the workgroups' in k_wgrad_sum, in order.
// A row of dy that is not finite must not meet the zeros of absent neighbours: such batches, found by their exponents, clear
// the rows that an offset does not have.
struct WgradMapParams {
  const void* feats;  // [n_in][C_in]
  const void* dout;   // [n_out][C_out]
  const int* map;     // [rows_pad][V]
  float* partial;     // [group][V][C_in][C_out]
  unsigned feats_bytes, dout_bytes, map_bytes;
  int C_in, C_out, V;
  int batches;        // of 32 rows
};

template <int TI, int TO, int J> struct WgradMapShape {
  static constexpr int BP = 32, NW = 8;
  static constexpr int x_bytes = BP * TI * 2, d_bytes = BP * TO * 2;
  static constexpr int LX = x_bytes / 1024, LD = d_bytes / 1024, LM = (J * BP + 63) / 64;  // loads of a unit, of dy, of the map
  static constexpr int map_bytes = LM * 256;
  static constexpr int wave_bytes = J * x_bytes + d_bytes + 2 * map_bytes;
  static constexpr int sum_bytes = NW * TI * TO * 4;
  static constexpr int total = NW * wave_bytes > sum_bytes ? NW * wave_bytes : sum_bytes;
  // Loads that may be in flight when unit j of a batch is read.  A step j issues unit j - 1 of the next batch (step 0: the last one
  // of its own), step 1 after that dy of the next batch and the map of the one after it.
  static constexpr int in_flight(int j) {
    int n = (J - 2) * LX;
    if (j == 0) return n;  // (dy and the map, issued in step 1, have landed as well)
    for (int d = 1; d < J; ++d)
      if ((j - d + J) % J == 1 % J) n += LD + LM;
    return n;
  }
  static_assert(J >= 3 && total <= 160 * 1024 && in_flight(J - 1) < 64, "");
};

template <typename F, int... I> __device__ __forceinline__ void for_constants(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

template <typename T, int TI, int TO, int J>
__global__ void __launch_bounds__(512) k_wgrad_map(const WgradMapParams p) {
  typedef WgradMapShape<TI, TO, J> W;
  constexpr int CX = TI / 8, CD = TO / 8, IB = TI / 16, OB = TO / 16, LX = W::LX, LD = W::LD, NW = W::NW, BP = W::BP;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fa = lane & 15, fg = lane >> 4;
  unsigned char* const my = smem + wave * W::wave_bytes;  // J units of x, dy, two maps
  const unsigned lds = (unsigned)(size_t)(__attribute__((address_space(3))) void*)my;
  constexpr int kD = J * W::x_bytes, kMap = kD + W::d_bytes;
  const int k0 = blockIdx.y * J, nk = min(J, p.V - k0);
  const int first = blockIdx.x * NW + wave, step = gridDim.x * NW;
  const int mine = p.batches > first ? (p.batches - first + step - 1) / step : 0;

  const u32x4 x_rsrc = rsrc_of(p.feats, p.feats_bytes), d_rsrc = rsrc_of(p.dout, p.dout_bytes), m_rsrc = rsrc_of(p.map, p.map_bytes);
  const unsigned x_row = (unsigned)p.C_in * 2u, d_row = (unsigned)p.C_out * 2u;
  int x_lane_row[LX];
  unsigned x_off[LX], d_off[LD];
#pragma unroll
  for (int i = 0; i < LX; ++i) {
    const int q = i * 64 + lane, r = q / CX, c = q % CX, ch = (block_at<2, CX>(c / 2, r) * 2 + c % 2) * 8;
    x_lane_row[i] = r;
    x_off[i] = ch < p.C_in ? (unsigned)ch * 2u : kNoRow;
  }
#pragma unroll
  for (int i = 0; i < LD; ++i) {
    const int q = i * 64 + lane, r = q / CD, c = q % CD, ch = (block_at<2, CD>(c / 2, r) * 2 + c % 2) * 8;
    d_off[i] = ch < p.C_out ? (unsigned)r * d_row + (unsigned)ch * 2u : kNoRow;
  }
  unsigned xa[IB], da[OB];  // fragment addresses
  {
    const int r = 8 * fg + (fa >> 2), in = (fa & 3) * 8;
#pragma unroll
    for (int i = 0; i < IB; ++i) xa[i] = (unsigned)(r * TI * 2 + place_of<2, CX>(i, r) * 32 + in);
#pragma unroll
    for (int o = 0; o < OB; ++o) da[o] = (unsigned)(kD + r * TO * 2 + place_of<2, CD>(o, r) * 32 + in);
  }
  auto frag = [&](const unsigned char* at, int pitch) -> u32x4 {  // (see k_wgrad)
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at + 4 * pitch));
    return __builtin_bit_cast(u32x4, s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
  };

  auto load_map = [&](int i) {  // entries [offset][row] of own batch i
    const bool live = i < mine;
    const unsigned row0 = (unsigned)(first + i * step) * BP;
#pragma unroll
    for (int l = 0; l < W::LM; ++l) {
      const int e = l * 64 + lane, r = e % BP, j = e / BP;
      load_dword_to_lds(m_rsrc, live && j < nk ? ((row0 + (unsigned)r) * (unsigned)p.V + (unsigned)(k0 + j)) * 4u : kNoRow,
                        lds + kMap + (i & 1) * W::map_bytes + l * 256);
    }
  };
  auto load_d = [&](int i) {
    const bool live = i < mine;
    const unsigned at = (unsigned)(first + i * step) * BP * d_row;
#pragma unroll
    for (int l = 0; l < LD; ++l) load_to_lds(d_rsrc, live && d_off[l] != kNoRow ? at + d_off[l] : kNoRow, 0, lds + kD + l * 1024);
  };
  unsigned src[LX];
  auto read_idx = [&](int i, int j) {  // where unit j of own batch i gathers from
    const unsigned char* at = my + kMap + (i & 1) * W::map_bytes + j * (BP * 4);
    const bool live = i < mine && j < nk;
    unsigned row[LX];
#pragma unroll
    for (int l = 0; l < LX; ++l) row[l] = *reinterpret_cast<const unsigned*>(at + x_lane_row[l] * 4);
#pragma unroll
    for (int l = 0; l < LX; ++l)  // (an absent neighbour, -1, wraps to just below 2^32)
      src[l] = live && x_off[l] != kNoRow ? row[l] * x_row + x_off[l] : kNoRow;
  };
  auto load_x = [&](int j) {
#pragma unroll
    for (int l = 0; l < LX; ++l) load_to_lds(x_rsrc, src[l], 0, lds + j * W::x_bytes + l * 1024);
  };

  f32x4 acc[J][OB][IB];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int o = 0; o < OB; ++o)
#pragma unroll
      for (int i = 0; i < IB; ++i) acc[j][o][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  load_map(0);
  load_map(1);
  load_d(0);
  wait_loads<0>();
#pragma unroll
  for (int j = 0; j < J - 1; ++j) {
    read_idx(0, j);
    load_x(j);
  }
  read_idx(0, J - 1);
  for (int b = 0; b < mine; ++b) {
    u32x4 d[OB];
    bool odd = false;  // some element of dy is not finite
    auto unit = [&](auto index) {
      constexpr int j = decltype(index)::value;
      wait_loads<W::in_flight(j)>();
      if (j == 0) {
#pragma unroll
        for (int o = 0; o < OB; ++o) d[o] = frag(my + da[o], TO * 2);
      }
      u32x4 x[IB];
#pragma unroll
      for (int i = 0; i < IB; ++i) x[i] = frag(my + j * W::x_bytes + xa[i], TI * 2);
      load_x(j == 0 ? J - 1 : j - 1);
      if (j == 1) {
        load_d(b + 1);
        load_map(b + 2);
      }
      read_idx(b + 1, j);
      if (j == 0) {  // an exponent of ones carries into the sign's place
        constexpr unsigned kExp = sizeof(T) == 2 && __is_same(T, _Float16) ? 0x7C007C00u : 0x7F807F80u;
        constexpr unsigned kOne = __is_same(T, _Float16) ? 0x04000400u : 0x00800080u;
        unsigned m = 0;
#pragma unroll
        for (int o = 0; o < OB; ++o)
#pragma unroll
          for (int q = 0; q < 4; ++q) m |= (d[o][q] & kExp) + kOne;
        odd = __any((m & 0x80008000u) != 0);
      }
      if (!odd) {
#pragma unroll
        for (int o = 0; o < OB; ++o)
#pragma unroll
          for (int i = 0; i < IB; ++i) acc[j][o][i] = mma<T>(d[o], x[i], acc[j][o][i]);
      } else {
        unsigned keep[4] = {0, 0, 0, 0};  // rows 8 fg .. 8 fg + 7, two to a word
        if (j < nk)
          for (int r = 0; r < 8; ++r) {
            const long long row = (long long)(first + b * step) * BP + 8 * fg + r;
            if (p.map[row * p.V + k0 + j] >= 0) keep[r >> 1] |= 0xFFFFu << (16 * (r & 1));
          }
#pragma unroll
        for (int o = 0; o < OB; ++o) {
          const u32x4 dk = {d[o][0] & keep[0], d[o][1] & keep[1], d[o][2] & keep[2], d[o][3] & keep[3]};
#pragma unroll
          for (int i = 0; i < IB; ++i) acc[j][o][i] = mma<T>(dk, x[i], acc[j][o][i]);
        }
      }
    };
    for_constants(unit, std::make_integer_sequence<int, J>{});
  }
  wait_loads<0>();  // (nothing may land in LDS that is used for something else next)
  f32x4* sums = reinterpret_cast<f32x4*>(smem);  // [wave][block][lane]
  constexpr int B = OB * IB;
  for (int j = 0; j < nk; ++j) {
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < J; ++jj)
      if (jj == j) {
#pragma unroll
        for (int o = 0; o < OB; ++o)
#pragma unroll
          for (int i = 0; i < IB; ++i) sums[(wave * B + o * IB + i) * 64 + lane] = acc[jj][o][i];
      }
    __syncthreads();
    float* dst = p.partial + ((long long)blockIdx.x * p.V + k0 + j) * p.C_in * p.C_out;
    for (int blk = wave; blk < B; blk += NW) {
      f32x4 v = sums[blk * 64 + lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += sums[(w * B + blk) * 64 + lane];
      const int o = blk / IB, i = blk % IB, ci = i * 16 + fa, co = o * 16 + fg * 4;
      if (ci < p.C_in && co < p.C_out) *reinterpret_cast<f32x4*>(dst + (long long)ci * p.C_out + co) = v;
    }
  }
}

// dW[e] = sum over the groups, in order: four waves take every fourth group, their sums are added in wave order.
__global__ void __launch_bounds__(256) k_wgrad_sum(const float* __restrict__ partial, int groups, long long elems, float* __restrict__ dw) {
  __shared__ float4 part[4][64];
  const int col = threadIdx.x & 63, stripe = threadIdx.x >> 6;
  const long long e4 = ((long long)blockIdx.x * 64 + col) * 4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (e4 < elems) {
    for (int g0 = stripe; g0 < groups; g0 += 32) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        v[u] = g0 + 4 * u < groups ? *reinterpret_cast<const float4*>(partial + (g0 + 4 * u) * elems + e4) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s.x += v[u].x;
        s.y += v[u].y;
        s.z += v[u].z;
        s.w += v[u].w;
      }
    }
  }
  part[stripe][col] = s;
  __syncthreads();
  if (stripe == 0 && e4 < elems) {
    float4 t = part[0][col];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      t.x += part[w][col].x;
      t.y += part[w][col].y;
      t.z += part[w][col].z;
      t.w += part[w][col].w;
    }
    *reinterpret_cast<float4*>(dw + e4) = t;
  }
}

}  // namespace

// Tiles by channels: as wide as the layer, so that a pair's rows are gathered once.  Beyond 128 channels only
// where there are pairs enough: a 256 x 256 tile is one workgroup per CU, with a partial tile of 256 KB each (85k pairs,
// 256 -> 256: 128 x 128 tiles 37 us, of which 6 for the reduction), or tiles so many that they fill the GPU anyway (421k
// pairs 768 -> 768: 717 us, 128 x 128 tiles 1005 us; 38k pairs: 132, 129).  weight: sqrt(time of a pair / time of a partial tile), from
// sweeps of the piece length (60k-row scan 128 -> 128, 512 / 1024 / 2048 pairs: 40 / 35 / 36 us; 100k rows
// 64 -> 64, 1024 / 2048 / 4096: 27 / 22 / 23 us).  32-wide tiles stay within one round (2.7M pairs 32 -> 32: 75 us, in two
// rounds 78; 271k pairs: 10.8, 12.3).
#define SPC_WGRAD_16(X) X(32, 32, 1, 1, 4, 4) X(64, 64, 1, 1, 4, 3) X(96, 96, 2, 2, 1, 3) X(128, 128, 2, 2, 1, 3) X(256, 256, 2, 4, 1, 4)
#define SPC_WGRAD_32(X) X(32, 32, 1, 1, 4, 3) X(64, 64, 1, 1, 4, 2)

namespace {
struct TilePick {
  int tile, per_cu;
  float weight;
};
TilePick pick_tile(int C_in, int C_out, bool f32, int64_t pairs) {
  const int c = std::max(C_in, C_out);
  if (f32) return c <= 32 ? TilePick{32, 2, 1.1f} : TilePick{64, 2, 0.9f};
  if (c <= 32) return {32, 1, 1.1f};
  if (c <= 64) return {64, 1, 0.75f};
  if (c <= 96) return {96, 3, 0.65f};
  // (a 256-wide tile of a layer with one narrow side multiplies mostly padding: 2.7M pairs 16 -> 256 367 us, with 128 x
  // 128 tiles 280; 64 -> 256 381 and 304; 96 -> 256 373 and 386)
  if (c <= 128 || std::min(C_in, C_out) <= 64 || (c <= 384 && pairs < (1 << 19))) return {128, 3, 0.6f};
  return {256, 1, 0.4f};
}
// As many pieces as the GPU holds at once, where that leaves each offset a few: wide layers have so many tiles that every
// piece comes in several rounds anyway, and one piece per offset would wait for the longest one (421k pairs, of
// which a quarter at the centre offset: fp32 256 -> 256 1650 us at one piece per offset, 548 us at 2,900 pairs a piece;
// f16 640 -> 640 1528 and 635 us).
Split split_for(const TilePick& t, int64_t tiles, int V, int64_t pairs) {
  Split s{};
  s.weight = t.weight / sqrtf((float)tiles);
  s.unit = 64;
  s.per_round = (int)std::max<int64_t>(1, 256 / tiles);
  const int64_t at_once = 256 * t.per_cu / tiles;
  int64_t g = std::min<int64_t>((int64_t)(s.weight * sqrt((double)pairs)) + 2, ceil_div(pairs, s.unit));
  if (at_once >= 3 * V) g = std::min<int64_t>(g, at_once - V);
  g = std::max<int64_t>(g, 1);
  s.pieces = (int)g + V;
  return s;
}
template <typename T, int TI, int TO, int NWI, int NWO, int NWK, int S>
int launch_wgrad(const WgradParams& p, dim3 grid, hipStream_t st) {
  typedef WgradShape<T, TI, TO, NWI, NWO, NWK, S> W;
  static_assert(W::total <= 160 * 1024, "LDS of a CU");
  auto kernel = k_wgrad<T, TI, TO, NWI, NWO, NWK, S>;
  static std::atomic<bool> attr_set{false};  // (set twice by racing threads at worst: the calls are idempotent)
  if (!attr_set.load(std::memory_order_acquire)) {
    SPC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, W::total));
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kernel, grid, dim3(W::threads), W::total, st, p);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}
}  // namespace

namespace {
constexpr int kMapChannels = 32, kMapOffsets = 7;  // of a k_wgrad_map tile and wave
template <typename T> int launch_wgrad_map(const WgradMapParams& p, dim3 grid, hipStream_t st) {
  typedef WgradMapShape<kMapChannels, kMapChannels, kMapOffsets> W;
  auto kernel = k_wgrad_map<T, kMapChannels, kMapChannels, kMapOffsets>;
  static std::atomic<bool> attr_set{false};  // (set twice by racing threads at worst: the calls are idempotent)
  if (!attr_set.load(std::memory_order_acquire)) {
    SPC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, W::total));
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kernel, grid, dim3(W::NW * 64), W::total, st, p);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}
}  // namespace

// Whether a call without a piece length takes its gradient straight from the map: narrow layers on maps that were known to have
// many pairs, and many per row, when the kmap's first such call was made.  Over pairs and from the map, us, f16, once the list is
// there (a first call over pairs makes it, 14 to 25 us more; it serves every layer on the kmap and fetch-on-demand):
//   pairs   0.53M        0.74M         0.91M         1.13M       1.28M (uniform)  1.44M       1.69M (uniform)  2.8M
//   16->16  12.6, 16.7   14.9, 18.5    18.4, 21.7    22.2, 23.4  20.5, 23.2       28.7, 27.0  28.1, 26.8       60.5, 49.6
//   32->32  15.8, 18.5   21.2, 20.6    27.8, 24.7    31.8, 27.8  31.2, 28.2       42.0, 33.6  40.7, 35.5       80.8, 64.1
//   8->32   13.0, 16.6   15.6, 18.3    18.6, 21.1    21.2, 22.9  21.4, 23.0       29.0, 26.2  27.2, 25.9       65.4, 41.5
//   32->8   12.9, 16.8   15.6, 18.2    19.8, 21.8    25.0, 24.8  23.3, 25.4       31.1, 30.8  31.1, 32.5       59.2, 59.0
// The line lies where the kernels alone are about equal, so that layers which share a list lose nothing to speak of; one narrow layer
// on a map of its own would gain from 0.3M pairs on (34 with the list, 15).
bool wgrad_from_map(const spconv_kmap* km, int C_in, int C_out, spconv_dtype dtype) {
  if (dtype == SPCONV_F32 || C_in > kMapChannels || C_out > kMapChannels || km->V != 27) return false;
  if (km->wgrad_known_pairs < 1200000 || km->wgrad_known_pairs < 7 * km->n_out) return false;
  return (uint64_t)km->n_in * C_in * 2 < kNoRow && (uint64_t)km->n_out * C_out * 2 < kNoRow &&
         (uint64_t)km->out_side.rows_pad * km->V * 4 < kNoRow;  // buffer descriptors address 32 bits
}

int wgrad_map_run(spconv_kmap* km, const void* feats, const void* dout, int C_in, int C_out, spconv_dtype dtype, float* dweights, hipStream_t st) {
  const int V = km->V, types = (int)ceil_div(V, kMapOffsets), groups = 256 / types;  // one workgroup per CU
  WgradMapParams p{};
  const long long elems = (long long)V * C_in * C_out;
  SPC_TRY(km->scratch.reserve((size_t)groups * elems * sizeof(float)));
  p.feats = feats;
  p.dout = dout;
  p.map = km->out_side.map.as<int>();
  p.partial = km->scratch.as<float>();
  p.feats_bytes = (unsigned)((uint64_t)km->n_in * C_in * 2);
  p.dout_bytes = (unsigned)((uint64_t)km->n_out * C_out * 2);
  p.map_bytes = (unsigned)((uint64_t)km->out_side.rows_pad * V * 4);
  p.C_in = C_in;
  p.C_out = C_out;
  p.V = V;
  p.batches = (int)ceil_div(km->n_out, 32);  // (the map is padded to whole batches)
  const dim3 grid((unsigned)groups, (unsigned)types);
  SPC_TRY(dtype == SPCONV_F16 ? launch_wgrad_map<_Float16>(p, grid, st) : launch_wgrad_map<__bf16>(p, grid, st));
  hipLaunchKernelGGL(k_wgrad_sum, dim3((unsigned)ceil_div(elems / 4, 64)), dim3(256), 0, st, p.partial, groups, elems, dweights);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

// Pairs of a piece that calls without a configuration get.
int64_t wgrad_auto_pairs(const spconv_kmap* km, int C_in, int C_out, spconv_dtype dtype) {
  const int64_t pairs = std::max<int64_t>(km->n_pairs, 1);
  const TilePick t = pick_tile(C_in, C_out, dtype == SPCONV_F32, pairs);
  const Split s = split_for(t, ceil_div(C_in, t.tile) * ceil_div(C_out, t.tile), km->V, pairs);
  return std::max<int64_t>(s.unit, ceil_div(pairs, s.pieces - km->V));
}

// piece_pairs: pairs of a piece, 0: chosen here.
int wgrad_run(spconv_kmap* km, const PairList& pl, int64_t piece_pairs, const void* feats, const void* dout, int C_in, int C_out,
              spconv_dtype dtype, float* dweights, hipStream_t st) {
  const int V = km->V;
  const int elems = C_in * C_out;
  const size_t e = dtype == SPCONV_F32 ? 4 : 2;
  const uint64_t feats_bytes = (uint64_t)km->n_in * C_in * e, dout_bytes = (uint64_t)km->n_out * C_out * e;
  const uint64_t pairs_bytes = (uint64_t)round_up(std::max<int64_t>(pl.cap, 0), 2) * 8;
  const bool fits = feats_bytes < kNoRow && dout_bytes < kNoRow && pairs_bytes < kNoRow;  // buffer descriptors address 32 bits
  if (dtype != SPCONV_F32 && !fits) return SPCONV_EINVAL;
  WgradParams p{};
  const TilePick t = pick_tile(C_in, C_out, dtype == SPCONV_F32, pl.cap);
  const int tile = dtype == SPCONV_F32 && !fits ? 64 : t.tile;
  if (piece_pairs > 0) {  // about 2^20 pieces at most: a smaller request is raised
    constexpr int64_t kMaxPieces = 1 << 20;
    p.split.length = (int)std::min<int64_t>(std::max<int64_t>(piece_pairs, ceil_div(pl.cap, kMaxPieces)), 1 << 30);
    p.split.pieces = (int)ceil_div(pl.cap, p.split.length) + V;
  } else {
    p.split = split_for(t, ceil_div(C_in, tile) * ceil_div(C_out, tile), V, pl.cap);
  }
  SPC_TRY(km->scratch.reserve((size_t)p.split.pieces * elems * sizeof(float)));
  p.feats = feats;
  p.dout = dout;
  p.pairs = pl.pairs.as<int2>();
  p.seg = pl.seg.as<int>();
  p.partial = km->scratch.as<float>();
  p.feats_bytes = (unsigned)feats_bytes;
  p.dout_bytes = (unsigned)dout_bytes;
  p.pairs_bytes = (unsigned)pairs_bytes;
  p.C_in = C_in;
  p.C_out = C_out;
  p.V = V;
  if (pl.cap > 0) {
    const dim3 grid((unsigned)p.split.pieces, (unsigned)ceil_div(C_in, tile), (unsigned)ceil_div(C_out, tile));
    if (dtype == SPCONV_F32 && !fits) {
      hipLaunchKernelGGL(k_wgrad_f32, grid, dim3(256), 0, st, p);
      SPC_LAUNCH_CHECK();
    } else {
      int status = SPCONV_EINVAL;
#define SPC_WGRAD_F16(TI, TO, NWI, NWO, NWK, S) \
  if (tile == TI) status = launch_wgrad<_Float16, TI, TO, NWI, NWO, NWK, S>(p, grid, st);
#define SPC_WGRAD_BF16(TI, TO, NWI, NWO, NWK, S) \
  if (tile == TI) status = launch_wgrad<__bf16, TI, TO, NWI, NWO, NWK, S>(p, grid, st);
#define SPC_WGRAD_F32(TI, TO, NWI, NWO, NWK, S) \
  if (tile == TI) status = launch_wgrad<float, TI, TO, NWI, NWO, NWK, S>(p, grid, st);
      if (dtype == SPCONV_F16) {
        SPC_WGRAD_16(SPC_WGRAD_F16)
      } else if (dtype == SPCONV_BF16) {
        SPC_WGRAD_16(SPC_WGRAD_BF16)
      } else {
        SPC_WGRAD_32(SPC_WGRAD_F32)
      }
      SPC_TRY(status);
    }
  }
  dim3 rgrid((unsigned)ceil_div(elems / 4, 64), (unsigned)V);
  hipLaunchKernelGGL(k_wgrad_reduce, rgrid, dim3(256), 0, st, km->scratch.as<float>(), pl.seg.as<int>(), V, p.split,
                     elems, dweights);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

}  // namespace spc
