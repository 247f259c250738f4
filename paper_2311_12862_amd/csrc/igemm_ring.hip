// Implicit-GEMM forward / input-gradient with workgroup tiles (Sections 2.2.3, 3.1, 3.2, 4.1), operands
// loaded straight into LDS: wide layers, and every fp32 layer.
//
// A workgroup owns BM consecutive rows of the (usually mask-sorted) map and BN output channels and walks the
// units (offset, piece of the reduction) that some row of the tile has.  A unit's operands - one 64- or
// 128-byte piece of each of the BM gathered rows, and the matching piece of the weight slice - are fetched
// by buffer loads that write LDS (lane l to base + 16 l; an absent neighbour is an out-of-range offset
// and fills zeros), so a unit in flight costs no registers; two stages alternate, the next one fills while the
// matrix cores work on this one.  What was measured on the way (256 CUs): such loads deliver 88 B/ns per
// CU from L2 whether one or four are in flight per wave, 40 from the last-level cache, and pieces of 64
// bytes half of that beyond L2; three or four stages gain nothing over two, because the workgroups that
// their LDS displaces hide more latency than they do (100k rows 64 -> 64: 20.9 / 25.6 / 26.2 us with 2 / 3 / 4).
// What does bound small maps is the longest tile, one step after another: NWK groups of waves (two) therefore
// take every other unit of the same tile and add their sums at the end through LDS (9k rows, 256 -> 256: 58
// -> 41 us with two groups, 37 us with 32-row tiles; 94 us for the register-staged kernel on the unsorted map).
// Beyond that, what a step takes is the CU's address unit (16 cycles per load of any wave) and waves that wait for each other at its
// barrier; where K groups are one wave each there is no barrier, and one wave's loads are issued while another multiplies: 9k rows,
// 256 -> 256, eight such groups on 64 x 64 tiles: 36 -> 24 us.
// Column tiles are dealt to the XCDs, so that each L2 holds one column tile of the weights (the same
// layer: 46 -> 37 us).
//
// LDS holds the pieces unpadded, as the loads write them; bank conflicts are avoided by the choice of which
// 16-byte chunk a lane fetches (XOR with the row, undone by the fragment reads).  The weights are the first operand
// of the matrix instructions: a lane then ends up with four consecutive output channels of one row,
// which it stores at once.
#include "common.h"
#include "lds_tiles.h"

#include <algorithm>
#include <atomic>

namespace spc {
namespace {

struct RingParams {
  const void* feats;
  const void* weights;
  void* out;
  float* partial;
  const int* map[kMaxSplit];
  const int* perm[kMaxSplit];
  const unsigned* blkmask[kMaxSplit];  // sorted plans: masks of 16-row blocks
  const unsigned* rowmask;             // unsorted plans: masks of rows
  int lo[kMaxSplit], width[kMaxSplit];
  long long rows;
  int V, c_red, c_out, C_in, C_out, mirror;
  int heavy_first;  // sorted maps: tiles late in the order hold the most offsets; they start first
  int n_tiles;
  int n_cols;       // column tiles where they are dealt to the XCDs (2, 4 or 8), or 1: grid y is the column tile
  unsigned feats_bytes, rows_pad;
};

constexpr unsigned kNoRow = 0xFFFF0000u, kNoWeight = 0x80000000u;  // out of range, also with a scalar offset added

// BM x BN outputs; PB bytes of a row per unit (64 or 128), E bytes per element, NW waves in all, NWK K groups for each of
// NWR such tiles, one below the other
// (256-row tiles of 64-byte pieces: four stages, see the alternating halves below)
template <int BM, int BN, int PB, int E, int NW, int NWK, int NWR> struct RingSmem {
  static constexpr int stages = BM == 256 && PB == 64 ? 4 : 2;
  static constexpr int a_bytes = BM * PB, b_bytes = PB / E * BN * E, unit = a_bytes + b_bytes, stage = NWR * NWK * unit;
  static constexpr int slab = (NWR * BM * 27 * 4 + NW * 1024 - 1) / (NW * 1024) * (NW * 1024);  // whole loads of every wave
  static constexpr int total = stages * stage + slab;
};

template <typename T, int BM, int BN, int PB, int NWM, int NWN, int NWK, int NWR, bool DGRAD>
__global__ void __launch_bounds__(NWM* NWN* NWK* NWR * 64) k_ring(const RingParams p) {
  constexpr int E = (int)sizeof(T), CE = 16 / E, KC = PB / E;  // bytes and chunk length of an element, channels of a unit
  constexpr int NW = NWM * NWN;                                // waves of a K group
  typedef RingSmem<BM, BN, PB, E, NW * NWK * NWR, NWK, NWR> L;
  constexpr int WM = BM / NWM, WN = BN / NWN, MB = WM / 16, NB = WN / 16;
  constexpr int CPR = PB / 16;              // chunks of a gathered piece
  constexpr int RPI = 64 / CPR;             // rows that one load covers
  constexpr int NA = BM / RPI / NW;         // gather loads per wave and unit
  constexpr int NBI = L::b_bytes / 1024;    // weight loads per unit
  constexpr int NBW = (NBI + NW - 1) / NW;  // per wave (with fewer than NW, some waves load the same piece)
  constexpr int LPR = DGRAD ? CPR : BN / CE;  // chunks of a row of the weight tile
  constexpr int RPB = 64 / LPR;               // rows of it per load
  static_assert((NWK & (NWK - 1)) == 0 && (NWK <= 2 || NW == 1) && (NWR == 1 || NWR == 2), "first_piece, units_of, tmask_other");
  static_assert(NW > 1 || (NWR == 1 && MB * NB % NWK == 0), "the waves share the sums");
  static_assert(NA >= 1 && BM % (RPI * NW) == 0 && NBI >= 1 && (NBI % NW == 0 || NW % NBI == 0), "whole loads per wave");
  extern __shared__ __align__(16) unsigned char smem[];
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  const int* mapS = reinterpret_cast<const int*>(smem + L::stages * L::stage);

  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = wave_all % NW, unit = wave_all / NW;                 // within its tile and K group, and which of these
  const int grp = NWK > 1 ? unit % NWK : 0, half = NWR > 1 ? unit / NWK : 0;  // K group, tile of the workgroup
  const int wm = wave / NWN, wn = wave % NWN;
  const int fa = lane & 15, fg = lane >> 4;  // fragment row / column, and chunk of a sub-step
  const int part = blockIdx.z;
  int t_idx = blockIdx.x, c_idx = blockIdx.y;
  if (p.n_cols > 1) {  // (workgroups go to the XCDs round-robin by their linear index)
    const unsigned at = blockIdx.y * gridDim.x + blockIdx.x, e = at & 7;
    c_idx = (int)e % p.n_cols;
    t_idx = (int)(at >> 3) * (8 / p.n_cols) + (int)e / p.n_cols;  // (every (tile, column) once, also in a last row that is not full)
  }
  const int tile = p.heavy_first ? p.n_tiles - 1 - t_idx : t_idx;
  const int n0 = c_idx * BN;
  const int width = p.width[part], lo = p.lo[part];
  const long long row0 = (long long)tile * (BM * NWR);

  {  // map slab of the tile (consecutive ints) -> LDS; past the end of the map: zeros, never used
    const u32x4 m_rsrc = rsrc_of(p.map[part], (unsigned)((unsigned long long)p.rows_pad * width * 4));
    const unsigned bytes = (unsigned)(NWR * BM * width * 4), begin = (unsigned)(row0 * width) * 4u;
    for (unsigned o = wave_all * 1024; o < bytes; o += NW * NWK * NWR * 1024)
      load_to_lds(m_rsrc, begin + o + lane * 16, 0, lds0 + L::stages * L::stage + o);
  }
  unsigned bmask = 0;  // lane b < NWR * BM / 16: mask of the 16-row block b
  if (p.rowmask) {
    constexpr int MR = (NWR * BM + 63) / 64;
    unsigned m[MR];
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      const long long r = row0 + i * 64 + lane;
      m[i] = r < p.rows && i * 64 + lane < NWR * BM ? p.rowmask[r] : 0u;
    }
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      for (int o = 1; o < 16; o <<= 1) m[i] |= __shfl_xor(m[i], o);
      const unsigned t = __shfl(m[i], (lane & 3) * 16);
      if ((lane >> 2) == i) bmask = t;
    }
  } else if (lane < NWR * BM / 16 && row0 + lane * 16 < p.rows) {
    bmask = p.blkmask[part][row0 / 16 + lane];
  }
  static_assert(NWR * BM <= 256, "blocks of a workgroup: 16 lanes");
  unsigned tmask = bmask;  // of the tile, and of the workgroup's other one
  for (int o = 1; o < BM / 16; o <<= 1) tmask |= __shfl_xor(tmask, o);
  const unsigned tmask_other = NWR > 1 ? __builtin_amdgcn_readlane(tmask, (half ^ 1) * (BM / 16)) : 0u;
  tmask = __builtin_amdgcn_readlane(tmask, half * (BM / 16));
  unsigned blk[MB], wave_mask = 0;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    blk[mb] = __builtin_amdgcn_readlane(bmask, (half * NWM + wm) * MB + mb);
    wave_mask |= blk[mb];
  }
  int orow[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const long long g = row0 + half * BM + wm * WM + mb * 16 + fa;
    orow[mb] = p.perm[part] ? p.perm[part][g] : (g < p.rows ? (int)g : -1);
  }

  const int c_red = p.c_red;
  const unsigned row_bytes = (unsigned)c_red * E, slice = (unsigned)(p.C_in * p.C_out) * E;
  const u32x4 x_rsrc = rsrc_of(p.feats, p.feats_bytes);
  const u32x4 w_rsrc = rsrc_of(p.weights, (unsigned)p.V * slice);
  const int n_pieces = (c_red + KC - 1) / KC;

  // Which chunk stands where.  Gathered pieces (and the input gradient's weight rows): 16 lanes read 8 rows x 2
  // neighbouring chunks per pass.  Forward weight rows: 16-bit types, the transposing read's passes touch rows r..r+3
  // and r+8..r+11 at one pair of chunks; fp32, four rows 4 apart at 64 bytes each.
  auto swz_a = [](int row) { return PB == 128 ? (row & 7) : ((row >> 2) & 1) * 2; };
  auto swz_b = [](int row) {
    if (E == 4) return LPR > 4 ? (((row >> 2) & 3) << 2) & (LPR - 1) : 0;
    return BN == 32 ? ((row >> 3) & 1) << 1
           : BN == 64 ? (((row >> 1) & 1) << 1) | (((row >> 3) & 1) << 2) : ((row & 3) << 1) | (((row >> 3) & 1) << 3);
  };
  const int g_row = lane / CPR, g_chunk = (lane % CPR) ^ swz_a(g_row);  // (RPI is a multiple of 8)
  const int* g_map = mapS + (half * BM + wave * NA * RPI + g_row) * width;
  unsigned w_off[NBW];  // this lane's chunk of the weight tile: offset within a slice, and
  int w_red[NBW];       // its reduction channel within a piece (far beyond any where there is no such column)
#pragma unroll
  for (int i = 0; i < NBW; ++i) {
    const int j = NBI >= NW ? wave * NBW + i : wave % NBI;
    const int r = j * RPB + lane / LPR;
    if constexpr (DGRAD) {  // rows: produced channel ci, chunks along co
      const int ch = (lane % LPR) ^ swz_a(r), ci = n0 + r;
      w_red[i] = ci < p.C_in ? ch * CE : 0x40000000;
      w_off[i] = (unsigned)(ci * p.C_out + ch * CE) * E;
    } else {  // rows: reduction channel ci, chunks along the produced channel co
      const int ch = (lane % LPR) ^ swz_b(r), co = n0 + ch * CE;
      w_red[i] = co < p.C_out ? r : 0x40000000;
      w_off[i] = (unsigned)(r * p.C_out + co) * E;
    }
  }

  // The units of this K group: set bits c of the tile mask, each with its pieces, dealt to the groups by their number
  // c * n_pieces + piece.  Which group takes a unit depends on the unit alone, not on the tile: a row's sums do not depend
  // on the rows beside it.
  const unsigned odd_start = NWK > 1 && (n_pieces & 1) ? 1u : 0u;
  auto first_piece = [&](int c) { return (grp - c * n_pieces) & (NWK - 1); };
  struct Cursor {
    unsigned rem;
    int c, piece;
  };
  auto cursor_settle = [&](Cursor& q) {
    while (q.piece >= n_pieces && q.rem) {
      q.c = __ffs((int)q.rem) - 1;
      q.rem &= q.rem - 1;
      q.piece = first_piece(q.c);
    }
  };
  auto cursor_step = [&](Cursor& q) {
    q.piece += NWK;
    cursor_settle(q);
  };
  Cursor qi{tmask, 0, n_pieces};  // the unit that is loaded next
  cursor_settle(qi);
  Cursor qc = qi;  // the unit that is multiplied next
  auto units_of = [&](unsigned of, int g) {  // units of K group g of a tile with this mask
    if (NWK == 1) return __popc(of) * n_pieces;
    if (!odd_start) return __popc(of) * (n_pieces / 2);
    return __popc(of & 0x55555555u) * ((n_pieces + 1 - g) / 2) + __popc(of & 0xAAAAAAAAu) * ((n_pieces + g) / 2);
  };
  int idx[NA];     // map entries of the unit that is loaded next
  auto fetch_idx = [&]() {
#pragma unroll
    for (int i = 0; i < NA; ++i) idx[i] = g_map[i * RPI * width + qi.c];
  };
  auto load_unit = [&](int slot) {
    const int k = lo + qi.c, r0 = qi.piece * KC;
    const unsigned a_lds = lds0 + slot * L::stage + unit * L::unit, b_lds = a_lds + L::a_bytes;
    const unsigned w_soff = (unsigned)(p.mirror ? p.V - 1 - k : k) * slice + (unsigned)(DGRAD ? r0 : r0 * p.C_out) * E;
    const bool ok = r0 + g_chunk * CE < c_red;
#pragma unroll
    for (int i = 0; i < NA; ++i)  // (an absent neighbour, -1, wraps to just below 2^32)
      load_to_lds(x_rsrc, ok ? (unsigned)idx[i] * row_bytes + (unsigned)g_chunk * 16u : kNoRow, (unsigned)r0 * E,
                  a_lds + (wave * NA + i) * 1024);
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const int j = NBI >= NW ? wave * NBW + i : wave % NBI;
      load_to_lds(w_rsrc, w_red[i] + r0 < c_red ? w_off[i] : kNoWeight, w_soff, b_lds + j * 1024);
    }
    cursor_step(qi);
    fetch_idx();
  };

  f32x4 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment addresses within a unit
  constexpr int KS = PB / 64;  // sub-steps
  unsigned xf[KS], wf[DGRAD ? KS : NB];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const unsigned ch = (unsigned)((ks * 4 + fg) ^ swz_a(fa)) * 16u;
    xf[ks] = (unsigned)((wm * WM + fa) * PB) + ch;
    if constexpr (DGRAD) wf[ks] = (unsigned)(L::a_bytes + (wn * WN + fa) * PB) + ch;
  }
  if constexpr (!DGRAD) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if constexpr (E == 2) {
        const int r = 8 * fg + (fa >> 2), ch = (wn * WN + nb * 16 + 4 * (fa & 3)) >> 3;
        wf[nb] = (unsigned)(L::a_bytes + r * BN * E + ((ch ^ swz_b(r)) * 16) + (fa & 1) * 8);
      } else {
        const int r = 4 * fg, ch = (wn * WN + nb * 16 + fa) >> 2;
        wf[nb] = (unsigned)(L::a_bytes + r * BN * E + ((ch ^ swz_b(r)) * 16) + (fa & 3) * 4);
      }
    }
  }
  struct Frags {
    u32x4 w[NB], x[MB];
  };
  auto read_frags = [&](int slot, int ks, Frags& f) {
    const unsigned char* st = smem + slot * L::stage + unit * L::unit;
    u32x4(&w)[NB] = f.w;
    u32x4(&x)[MB] = f.x;
    {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        if constexpr (DGRAD) {
          w[nb] = *reinterpret_cast<const u32x4*>(st + wf[ks] + nb * 16 * PB);
        } else if constexpr (E == 2) {
          // 16 lanes fetch a 4 x 16 block of [ci][co] and each receives one column: 4 reduction channels of
          // its output channel; two reads give the lane's 8 (ci = 8 fg .. 8 fg + 7)
          const unsigned char* b = st + wf[nb] + ks * 32 * BN * E;
          const s16x4 l4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(b));
          const s16x4 h4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(b + 4 * BN * E));
          w[nb] = __builtin_bit_cast(u32x4, s16x8{l4[0], l4[1], l4[2], l4[3], h4[0], h4[1], h4[2], h4[3]});
        } else {
          const unsigned char* b = st + wf[nb] + ks * 16 * BN * E;
#pragma unroll
          for (int i = 0; i < 4; ++i) w[nb][i] = *reinterpret_cast<const unsigned*>(b + i * BN * E);
        }
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) x[mb] = *reinterpret_cast<const u32x4*>(st + xf[ks] + mb * 16 * PB);
    }
  };
  auto multiply = [&](int c, const Frags& f) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      if ((blk[mb] >> c) & 1u) {  // (the lock-step unit: a 16-row block without this offset is skipped)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mma<T>(f.w[nb], f.x[mb], acc[mb][nb]);
      }
  };

  wait_loads_and_sync();  // the slab is there
  fetch_idx();
  if constexpr (L::stages == 4) {
    // Two halves of the waves, one wave of each on every SIMD, take turns: in one slot the first half reads its fragments of a unit
    // and issues its share of the loads three units ahead while the second half multiplies, in the next slot the other way round.
    // A unit's loads have five slots to land (each wave waits for its own before the barrier into the slot in which the unit is
    // first read), and its stage is filled again two slots after both halves have read it.  Beyond the last unit loads are
    // still issued, out of range, so that the counts stay.  Measured (300k rows of a room, against two stages and all waves in step):
    // input gradient 256 -> 256 463 -> 428 us, 136 -> 200 387 -> 315, forward 136 -> 200 289 -> 271; bound by the rows that come from
    // beyond the L2 (4.3 GB through the CUs' address units).
    static_assert(NWK == 1 && NWR == 1 && KS == 1 && NWM == 2, "");
    constexpr int NL = NA + NBW;
    const int mine = units_of(tmask, 0);
    auto load_next = [&](int u) {
      if (u < mine) {
        load_unit(u & 3);
      } else {
#pragma unroll
        for (int i = 0; i < NL; ++i) load_to_lds(x_rsrc, kNoRow, 0, lds0 + (u & 3) * L::stage + (wave * NL + i) * 1024);
      }
    };
    Frags f;
    for (int u = 0; u < 3; ++u) load_next(u);
    if (wm == 0) {
      for (int u = 0; u < mine; ++u) {
        wait_loads_and_sync<2 * NL>();
        read_frags(u & 3, 0, f);
        load_next(u + 3);
        sync_lds();
        __builtin_amdgcn_s_setprio(1);
        multiply(qc.c, f);
        __builtin_amdgcn_s_setprio(0);
        cursor_step(qc);
      }
      wait_loads_and_sync();
    } else {
      wait_loads_and_sync<2 * NL>();
      for (int u = 0; u < mine; ++u) {
        sync_lds();
        read_frags(u & 3, 0, f);
        load_next(u + 3);
        wait_loads_and_sync<2 * NL>();
        __builtin_amdgcn_s_setprio(1);
        multiply(qc.c, f);
        __builtin_amdgcn_s_setprio(0);
        cursor_step(qc);
      }
      wait_own_loads();
    }
  } else if constexpr (NW == 1) {
    // every wave is a K group: nothing is shared until the end, so nothing is waited for but the wave's own loads, and one
    // wave's loads are issued while another multiplies
    bool more = qi.piece < n_pieces;
    if (more) load_unit(0);
    for (int slot = 0; more; slot ^= 1) {
      wait_own_loads();  // (the other stage was read before: its fragments are in registers)
      more = qi.piece < n_pieces;
      Frags f[KS];
      read_frags(slot, 0, f[0]);
      if (more) load_unit(slot ^ 1);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks > 0) read_frags(slot, ks, f[ks]);
        multiply(qc.c, f[ks]);
      }
      cursor_step(qc);
    }
  } else {
    const int mine = units_of(tmask, grp);
    int steps = mine;  // every wave passes as many barriers
    if (NWK > 1) steps = max(steps, units_of(tmask, grp ^ 1));
    if (NWR > 1) steps = max(steps, max(units_of(tmask_other, 0), NWK > 1 ? units_of(tmask_other, 1) : 0));
    if (mine > 0) load_unit(0);
    for (int it = 0; it < steps; ++it) {
      wait_loads_and_sync();  // this step's unit has landed, and everyone is done with the stage that is filled next
      if (it + 1 < mine) load_unit((it + 1) & 1);
      if (it < mine && ((wave_mask >> qc.c) & 1u)) {
        Frags f[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          read_frags(it & 1, ks, f[ks]);
          multiply(qc.c, f[ks]);
        }
      }
      cursor_step(qc);
    }
  }
  const int c_out = p.c_out;
  // a lane holds channels 4 fg + r of row fa of each block
  auto store = [&](int to, int col, f32x4 v4) {
    if (col >= c_out) return;
    if (p.partial) {
      *reinterpret_cast<f32x4*>(p.partial + ((long long)part * p.rows + to) * c_out + col) = v4;
    } else {
      typedef T out4 __attribute__((ext_vector_type(4)));
      out4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = (T)v4[r];
      *reinterpret_cast<out4*>(reinterpret_cast<T*>(p.out) + (long long)to * c_out + col) = v;
    }
  };
  if constexpr (NW == 1) {  // the waves' sums meet in LDS; each adds up a share of the blocks, in order
    static_assert(NWK * BM * BN * 4 <= 2 * L::stage, "the sums fit the stages");
    wait_loads_and_sync();
    f32x4* sums = reinterpret_cast<f32x4*>(smem);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) sums[(grp * MB * NB + mb * NB + nb) * 64 + lane] = acc[mb][nb];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < MB * NB / NWK; ++u) {
      const int blk = grp * (MB * NB / NWK) + u;
      f32x4 v = sums[blk * 64 + lane];
#pragma unroll
      for (int g = 1; g < NWK; ++g) v += sums[(g * MB * NB + blk) * 64 + lane];
      int to = orow[0];
#pragma unroll
      for (int mb = 1; mb < MB; ++mb) to = blk / NB == mb ? orow[mb] : to;
      if (to >= 0) store(to, n0 + (blk % NB) * 16 + fg * 4, v);
    }
    return;
  }
  if constexpr (NWK > 1) {  // the K groups' sums meet in LDS; group 0 adds them up in order and stores
    static_assert(NWR * (NWK - 1) * BM * BN * 4 <= 2 * L::stage, "the sums fit the stages");
    wait_loads_and_sync();
    f32x4* sums = reinterpret_cast<f32x4*>(smem);
    if (grp > 0) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) sums[(((half * (NWK - 1) + grp - 1) * NW + wave) * MB * NB + mb * NB + nb) * 64 + lane] = acc[mb][nb];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 0; g < NWK - 1; ++g)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] += sums[(((half * (NWK - 1) + g) * NW + wave) * MB * NB + mb * NB + nb) * 64 + lane];
  }

#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    if (orow[mb] < 0) continue;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) store(orow[mb], n0 + wn * WN + nb * 16 + fg * 4, acc[mb][nb]);
  }
}

template <typename T, int BM, int BN, int PB, int NWM, int NWN, int NWK, int NWR>
int launch_ring(const RingParams& p, bool dgrad, dim3 grid, hipStream_t st) {
  constexpr int NW = NWM * NWN * NWK * NWR;
  typedef RingSmem<BM, BN, PB, (int)sizeof(T), NW, NWK, NWR> L;
  static_assert(L::total <= 160 * 1024, "LDS of a CU");
  static std::atomic<bool> attr_set{false};  // (set twice by racing threads at worst: the calls are idempotent)
  auto fwd = k_ring<T, BM, BN, PB, NWM, NWN, NWK, NWR, false>;
  auto dgr = k_ring<T, BM, BN, PB, NWM, NWN, NWK, NWR, true>;
  if (!attr_set.load(std::memory_order_acquire)) {
    SPC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(fwd), hipFuncAttributeMaxDynamicSharedMemorySize, L::total));
    SPC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(dgr), hipFuncAttributeMaxDynamicSharedMemorySize, L::total));
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(dgrad ? dgr : fwd, grid, dim3(NW * 64), L::total, st, p);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

// the tile shapes that are built: BM, BN, waves along the rows, along the columns, K groups, tiles of a workgroup
#define SPC_RING_SHAPES_16(X) \
  X(32, 64, 1, 1, 4, 1) X(32, 64, 1, 1, 8, 1) X(32, 64, 1, 2, 2, 1) X(64, 32, 4, 1, 1, 1) X(64, 64, 1, 1, 8, 1) X(64, 64, 2, 2, 1, 1) \
  X(64, 64, 2, 2, 2, 1) X(64, 128, 2, 2, 1, 1) X(128, 128, 2, 2, 1, 1) X(256, 256, 2, 4, 1, 1)
#define SPC_RING_SHAPES_32(X) \
  X(32, 16, 2, 1, 2, 2) X(32, 32, 1, 2, 2, 2) X(64, 16, 4, 1, 1, 1) X(64, 32, 1, 1, 8, 1) X(64, 32, 4, 1, 1, 1) X(64, 64, 2, 2, 1, 1) X(64, 64, 2, 2, 2, 1)
// (eight K groups of 128-byte pieces do not fit in LDS, four are for layers of 64-byte pieces)
constexpr bool ring_built(int pb, int nwk) { return nwk < 4 || pb == 64; }

template <typename T, int PB> int launch_shape(const RingParams& p, bool dgrad, const RingShape& s, dim3 grid, hipStream_t st) {
#define SPC_RING_CASE(BM, BN, NWM, NWN, NWK, NWR) \
  if (s.bm == BM * NWR && s.bn == BN && s.nwk == NWK && s.nwr == NWR) if constexpr (ring_built(PB, NWK)) return launch_ring<T, BM, BN, PB, NWM, NWN, NWK, NWR>(p, dgrad, grid, st);
  if constexpr (sizeof(T) == 4) {
    SPC_RING_SHAPES_32(SPC_RING_CASE)
  } else {
    SPC_RING_SHAPES_16(SPC_RING_CASE)
  }
  return SPCONV_EINVAL;
}

size_t ring_lds_bytes(const RingShape& s, bool f32) {
#define SPC_RING_LDS(BM, BN, NWM, NWN, NWK, NWR)                                                                     \
  if (s.bm == BM * NWR && s.bn == BN && s.nwk == NWK && s.nwr == NWR)                                                                 \
    return s.piece == 128 ? (size_t)RingSmem<BM, BN, 128, E, NWM * NWN * NWK * NWR, NWK, NWR>::total                       \
                          : (size_t)RingSmem<BM, BN, 64, E, NWM * NWN * NWK * NWR, NWK, NWR>::total;
  if (f32) {
    constexpr int E = 4;
    SPC_RING_SHAPES_32(SPC_RING_LDS)
  } else {
    constexpr int E = 2;
    SPC_RING_SHAPES_16(SPC_RING_LDS)
  }
  return 0;
}

int ring_waves(const RingShape& s, bool f32) {
#define SPC_RING_WAVES(BM, BN, NWM, NWN, NWK, NWR) \
  if (s.bm == BM * NWR && s.bn == BN && s.nwk == NWK && s.nwr == NWR) return NWM * NWN * NWK * NWR;
  if (f32) {
    SPC_RING_SHAPES_32(SPC_RING_WAVES)
  } else {
    SPC_RING_SHAPES_16(SPC_RING_WAVES)
  }
  return 0;
}

}  // namespace

// Where eight K groups of one wave each take a 64 x 64 tile (16-bit types): small maps, whose launch is as long as the chain of
// the longest tile.  Sorted maps, us, before (32 x 64 or 64 x 64, two K groups) and with them: 9k rows 256 -> 256 36, 24 (564 workgroups);
// 5k 512 -> 512 65, 44; 7k 128 -> 256 20, 16; 12k 192 -> 192 30, 27; 20k 256 -> 128 35, 27; where the line lies: 15k 256 -> 256
// (940 workgroups) 38, 38; 12k 128 -> 256 (752) 21, 23; 20k 128 -> 128 (626) 21, 21; 30k 96 -> 96 (938) 25, 27.5.  32-row tiles
// where the map is so small that these are fewer than three per CU and pieces come in whole rounds (4k rows 256 -> 256 33, 23, with
// 32 rows 19).  Map order, one round of workgroups (kernel 1 before): 12k rows 64 -> 64 15, 11.4; 7k 128 -> 128 23, 16; 96 -> 96 17,
// 14; 12k 128 -> 64 22, 15; 20k 64 -> 64 (313) 15, 20; 2k scattered points, of one pair a row, 64 -> 64 8.8, 9.1.
bool wave_groups(int V, int n_split, int c_red, int c_out, int64_t wgs) {
  if (V < 25 || c_red < 64 || c_out < 32) return false;  // (few offsets: few units to share)
  return wgs <= (n_split == 0 ? 256 : c_red % 64 ? 600 : std::min(900, c_red * 7 / 2));
}

// Tile shape from the row count and the produced channels.  The largest tile that still gives a few workgroups per
// CU: a larger one gathers each row and loads each weight slice fewer times, but small maps are bound by the
// longest tile.  Measured on sorted maps (us): 300k rows 256 -> 256, (256, 256) 435, (128, 128) 480; 96 -> 96, (128, 128)
// 125, (64, 128) 134; 100k rows 64 -> 128, (64, 128) 30.3, (128, 128) 31.4; 128 -> 64, two K groups (64, 64) 30.2, one
// 35.2; 30k rows 128 -> 128, (64, 64) with two K groups 24.9, (64, 128) 37.9, (128, 128) 47; 9k rows 256 -> 256, (32,
// 64) with two K groups 36.9, (64, 64) 41.2, (64, 128) 67.
int igemm_ring_shape(int V, int n_split, int64_t rows, int64_t rows_src, int c_red, int c_out, bool f32, bool dgrad,
                     bool small_tiles, RingShape* s) {
  *s = RingShape{};
  const int q = f32 ? 4 : 8, e = f32 ? 4 : 2;
  if (rows < 1 || rows_src < 0 || c_red < q || c_out < q || c_red % q || c_out % q) return SPCONV_EINVAL;
  PlanShape ps;
  SPC_TRY(plan_shape(V, rows, n_split, 16, &ps));
  const uint64_t bytes = (uint64_t)rows_src * c_red * e;
  // 32-bit buffer offsets; "no row" and "no weight" stay out of range with a scalar offset of one row added
  if (bytes >= (uint64_t)kNoRow - 0x8000u || (uint64_t)ps.rows_pad * 27 * 4 >= 0xFFFF0000ull ||
      (uint64_t)V * c_red * c_out * e >= kNoWeight)
    return SPCONV_EINVAL;
  s->feats_bytes = (unsigned)bytes;
  auto wgs = [&](int bm, int bn) { return ceil_div(rows, bm) * ceil_div(c_out, bn) * ps.parts; };
  s->nwk = s->nwr = 1;
  if (f32) {
    // The matrix cores' fp32 rate makes a tile with all 27 offsets last: 64 x 64 outputs of 64 channels 23 us of a CU
    // on its own.  So a workgroup takes two tiles of 32 x 32 outputs, each with two K groups, unless there are workgroups
    // enough for the longest not to matter.  Measured on sorted maps (us; 64 x 64 with two K groups, two 32 x 32, 64 x 32):
    // 2k rows 16 -> 16 8.8 (64 x 16), two 32 x 16 6.6; 5k 64 -> 64 37, 26; 30k 64 -> 64 44, 29.5; 60k 64 -> 64
    // 48, 42; and where the line lies: 30k 96 -> 96 66, 62; 50k of a dense room 64 -> 64 57, 62; 60k 96 -> 96 103 (one K
    // group), 96; 100k 128 -> 128 165 (one), 178.
    // On smaller maps, the more so the longer the reduction, eight K groups of a wave each end sooner still: 5k rows 96 -> 96 38, 28; 15k 64 -> 64 28,
    // 20; 10k 32 -> 32 16, 13; 30k 96 -> 32 40, 27; where the line lies: 30k 64 -> 64 30, 33; 32 -> 32 24, 25; 60k 96 -> 96 104, 104.
    // One of them fits on a CU, so that the rounds add up: wide layers (without and with these groups, scan; room) lie, by workgroups,
    //   1,264  512 -> 512 5k rows 211, 167; 353, 311       1,504  256 -> 128 24k 160, 95; 198, 192; 512 -> 128 24k 314, 168; 387, 358
    //   3,008  256 -> 256 24k 222, 176; 342, 361           3,128  512 -> 128 50k 492, 330; 717, 740
    //   3,008  512 -> 512 12k 465, 494; 678, 730           3,008  1024 -> 256 24k 874, 585; 1360, 1310
    //   4,032  1024 -> 1024 8k 1179, 804; 1697, 1679       6,016  512 -> 512 24k 578, 695; 1222, 1368
    //   6,256  1024 -> 256 50k 1170, 1183; 2576, 2747      11,880  1024 -> 256 95k 2290, 2600; 4010, 4500
    // The line lies between these: up to it scans gain up to a half, and rooms, whose tiles are all long, lose 7 % at most.
    // Tiles of a dense room all have their 27 offsets, and are bound by the work, not by the longest: 62k rows (64 x 64 with two K
    // groups, two 32 x 32) 64 -> 64 66, 77; 96 -> 64 94, 110; a scan of as many 57, 53; 82, 78; 45k 57, 59; 80, 86; scan 48, 42; 67,
    // 60.  Unsorted 45k 32 -> 32 (64 x 32, two 32 x 32) 36, 42; 30k 29.5, 28.  Short reductions have little to share between the K
    // groups: sorted 40k 32 -> 64 (1,250 workgroups; 64 x 64 with two K groups, two 32 x 32) of a dense scan 27, 35, a room 28, 34; 30k (938)
    // 22.5, 19; 27, 25; 64 -> 32 (64 x 32, two 32 x 32) of a scan and a room 80k (1,250) 46, 38; 50, 51; 100k (1,563) 48, 45; 53, 58.
    s->bm = 64;
    s->bn = c_out <= 16 ? 16 : 32;
    s->piece = c_red <= 16 ? 64 : 128;
    // In map order all tiles are of about the same length, so that a second round of workgroups counts in full: sorted 30k rows 32 -> 64
    // (938 workgroups) gain, unsorted lose (uniform 10k rows, eight groups or pairs, 314: 22.6, 25; 24k, pairs, 750: 34, 43; planes of K = 5, 30k
    // 64 -> 64, 938: 279, 308), while one round gains most (8k, 250: 22, 13.4; 4.5k 64 -> 128, 280: 39, 31; planes of K = 5, 8k of a room, without groups, pairs, eight groups, 96 -> 96, 375, -, 232, 215;
    // 128 -> 128, 500, -, 285, 270).
    // 2x2x2 maps have short chains.  Pairs, by workgroups: 32 -> 64 242 9.7, 8.0; 276 9.8, 10.3; 752 14.7, 17.5; 64 -> 128 552 23.5,
    // 20.9; 636 24.2, 24.4; 964 19, 20.8; 96 -> 96 414 32, 21.5; 477 18.6, 22.4; 723 25.2, 27.8; 128 -> 64 376 25.3, 26.7; sorted, 938, 11.7,
    // 13.3; 128 -> 256 1,104 27, 20.
    const bool ordered = n_split > 0;
    const int eight_to = V < 25 || c_red <= 16 || c_out <= 16 ? 0 : ordered ? std::min(12 * c_red, 2560 + 2 * c_red) : c_red <= 32 ? 288 : 512;
    const int pairs_to = V < 25         ? (c_red <= 32 ? 257 : c_red < 128 || c_out <= 64 ? 600 : 1300)
                         : c_out <= 32  ? (c_red <= 32 || !ordered ? 600 : c_red <= 64 ? 1500 : 2000)
                         : !ordered     ? (c_red <= 32 ? 289 : 512)
                                        : (c_red <= 32 ? 1000 : 1400);
    if (small_tiles && wgs(64, 32) <= eight_to) {
      s->nwk = 8;
      s->piece = 64;
    } else if (small_tiles && wgs(64, s->bn) < pairs_to) {
      s->nwk = s->nwr = 2;
    } else if (c_out > 32) {
      s->bn = 64;
      if (small_tiles && wgs(64, 64) < 1024) s->nwk = 2;
    }
  } else {
    s->piece = (c_red % 64 == 0) ? 128 : 64;
    if (small_tiles && wave_groups(V, n_split, c_red, c_out, wgs(64, 64))) {
      s->bm = c_red % 256 == 0 && wgs(32, 64) <= 768 ? 32 : 64;
      s->bn = 64;
      s->nwk = 8;
      s->piece = 64;
    } else if (small_tiles && n_split > 0 && c_red > 64 && c_red % 64 && c_out > 32 && wgs(64, 64) <= (c_red < 128 ? 1000 : 1600)) {
      // 32-row tiles with four K groups of a wave each: where tiles are of unequal length.  64 x 64 with two K groups, and these (sparse scan;
      // uniform; dense scan; room), by workgroups of 64 x 64:
      //   844    96 -> 96 -; 24.1, 18.8; 27.0, 28.5; 28.3, 30.0      136 -> 72 -; 36.0, 25.6; 39.3, 36.0; 43.8, 41.1
      //   940    96 -> 96 23.5, 18.2; 24.2, 20.1; -; 28.1, 30.4      136 -> 72 35.1, 25.0; 36.0, 25.7; -; 43.6, 41.4
      //   1,094  96 -> 96 -; 24.6, 22.4; 32.2, 33.8; 32.5, 35.2      200 -> 128 -; 49.6, 34.9; 59.8, 59.6; 64.5, 63.3
      //   1,250  96 -> 96 -; 25.4, 25.1; 32.9, 36.3; 34.8, 39.7      200 -> 128 -; 50.7, 40.0; 63.2, 64.0; 68.6, 72.0
      //   1,410  96 -> 96 29.5, 27.7; 26.1, 27.3; -; 36.9, 42.8      200 -> 128 57.5, 44.5; 51.0, 43.1; -; 73.8, 78.7
      //   1,564  96 -> 96 26.9, 28.4; 26.9, 29.6; -; 43.1, 48.9      200 -> 128 53.6, 44.8; 52.0, 46.7; -; 85.4, 92.4
      s->bm = 32, s->bn = 64;
      s->nwk = 4;
    } else if (c_out <= 32) {
      s->bm = 64, s->bn = 32;
    } else if (c_out > 128 && wgs(256, 256) >= 768) {
      // (four stages of 64-byte pieces, whose halves of waves take turns, where the weights need no transposing reads: 300k rows
      // 256 -> 256 input gradient 463 -> 428 us, forward 470 -> 467; 220k rows of a scan 239 -> 238, 243 -> 264)
      s->bm = 256, s->bn = 256;
      if (dgrad) s->piece = 64;
    } else if (c_out > 64 && wgs(128, 128) >= 1024) {
      s->bm = 128, s->bn = 128;
    } else if (c_out > 64 && wgs(64, 128) >= 1024) {
      s->bm = 64, s->bn = 128;
    } else {
      // two K groups where the units of a tile are many (long reductions), one where they are few
      s->bm = 64, s->bn = 64;
      s->nwk = c_red > 64 ? 2 : 1;
      if (s->nwk == 2 && wgs(64, 64) < 768 && small_tiles) s->bm = 32;
    }
  }
  s->threads = 64 * ring_waves(*s, f32);
  s->lds_bytes = ring_lds_bytes(*s, f32);
  s->n_tiles = ceil_div(rows, s->bm);
  const int64_t cols = ceil_div(c_out, s->bn);
  s->n_cols = cols == 2 || cols == 4 || cols == 8 ? (int)cols : 1;
  s->grid[0] = (unsigned)s->n_tiles;
  s->grid[1] = (unsigned)cols;
  s->grid[2] = (unsigned)ps.parts;
  return SPCONV_OK;
}

int igemm_ring_run(const spconv_kmap* km, const SideMap& side, const IgemmPlan& plan, const IgemmArgs& a, const RingShape& s,
                   hipStream_t st) {
  if (plan.rows == 0) return SPCONV_OK;
  RingParams p{};
  p.feats = a.feats;
  p.weights = a.weights;
  p.out = a.out;
  p.partial = a.partial;
  p.rows = plan.rows;
  p.V = km->V;
  p.C_in = a.C_in;
  p.C_out = a.C_out;
  p.mirror = a.mirror;
  p.c_red = a.dgrad ? a.C_out : a.C_in;
  p.c_out = a.dgrad ? a.C_in : a.C_out;
  p.feats_bytes = s.feats_bytes;
  p.rows_pad = (unsigned)plan.rows_pad;
  const int64_t tiles_alloc = std::max<int64_t>(plan.n_tiles, 1);
  for (int i = 0; i < plan.parts; ++i) {
    p.lo[i] = plan.lo[i];
    p.width[i] = plan.width[i];
    if (plan.n_split == 0) {
      p.map[i] = side.map.as<int>();
      p.rowmask = side.mask.as<unsigned>();
    } else {
      p.blkmask[i] = plan.tilemask.as<unsigned>() + (size_t)i * tiles_alloc;
      p.map[i] = plan.maps.as<int>() + plan.map_off[i];
      p.perm[i] = plan.perm.as<int>() + (size_t)i * plan.rows_pad;
    }
  }
  p.heavy_first = plan.n_split > 0;
  p.n_tiles = (int)s.n_tiles;
  p.n_cols = s.n_cols;
  const dim3 grid(s.grid[0], s.grid[1], s.grid[2]);
  const bool dgrad = a.dgrad != 0, wide = s.piece == 128;
  switch (a.dtype) {
    case SPCONV_F16: return wide ? launch_shape<_Float16, 128>(p, dgrad, s, grid, st) : launch_shape<_Float16, 64>(p, dgrad, s, grid, st);
    case SPCONV_BF16: return wide ? launch_shape<__bf16, 128>(p, dgrad, s, grid, st) : launch_shape<__bf16, 64>(p, dgrad, s, grid, st);
    case SPCONV_F32: return wide ? launch_shape<float, 128>(p, dgrad, s, grid, st) : launch_shape<float, 64>(p, dgrad, s, grid, st);
  }
  return SPCONV_EINVAL;
}

}  // namespace spc
