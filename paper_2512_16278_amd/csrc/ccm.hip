// Per-cell exact sums of Eq. 1 (Sec. 3.2): S_a = sum_t x_a(t) and
// S_ab = sum_t x_a(t) x_b(t), a <= b, for every (sub-interval, channel) cell.
//
// Main engine (ccm_mfma_kernel): the cell's beams x time samples form a small
// integer matrix X and the sums are X X^T, a dense contraction over time. The
// kernel feeds it to the int8 matrix cores (v_mfma_i32_16x16x32_i8) on
// x' = x - 128 (a byte XOR with 0x80), which is exact; the offset is removed
// again in integer arithmetic:
//     S_a  = S'_a + 128 L
//     S_ab = S'_ab + 128 (S'_a + S'_b) + 16384 L.
// S'_a comes out of the same products: one padding row of X is all ones.
//
// Data path: a workgroup owns CW consecutive channels of one sub-interval and
// walks its L samples in chunks of 32 rows. A chunk of every beam (32 rows x
// CW channel bytes) goes from HBM straight into LDS with the direct
// global-to-LDS loads (global_load_lds_dwordx4: lane l of a wave instruction
// fills bytes [16 l, 16 l + 16) of a 1 KB LDS window), into a ring of NST
// chunk buffers, so NST - 1 chunks are in flight while one is consumed and no
// registers hold staged data. The 16-byte units of a chunk are XOR-swizzled
// (unit ^= (beam + 2 (row / 8)) mod 8) so that the 64 lanes reading one row
// dword of 16 beams x 4 row groups hit every LDS bank group equally. A wave
// reads the rows of its channels back as dwords (4 channels x 1 time),
// transposes 4x4 bytes in registers (v_perm) to time-packed operands, and
// issues one MFMA per (channel, 16x16 beam block pair). Launches that fill the
// chip at 16 k to 16 k + 8 beams take the packed engine instead (takes_pack). Waits on the DMA use
// explicit vmcnt counts (every wave issues the same number of loads per
// chunk), not the workgroup fence, so later chunks stay in flight across the
// per-chunk barrier. The workgroups of 1 KB of adjacent channels are
// dispatched back to back on one XCD, so the rows are fetched in long runs.
//
// Comparison engine (ccm_valu_kernel, nbeam <= 20): one lane per channel, all
// pair accumulators in registers, four samples per v_dot4_u32_u8.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace rfi {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int TC = 32;              // rows per chunk = K of one MFMA
constexpr uint32_t OFFSET_XOR = 0x80808080u;

__device__ __forceinline__ void transpose4x4(uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3,
                                             uint32_t& o0, uint32_t& o1, uint32_t& o2,
                                             uint32_t& o3) {
  // rows r_i hold bytes (channel 0..3) of time i; o_c holds bytes (time 0..3)
  // of channel c.
  uint32_t t0 = __builtin_amdgcn_perm(r1, r0, 0x05010400u);
  uint32_t t1 = __builtin_amdgcn_perm(r3, r2, 0x05010400u);
  uint32_t t2 = __builtin_amdgcn_perm(r1, r0, 0x07030602u);
  uint32_t t3 = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
  o0 = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
  o1 = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
  o2 = __builtin_amdgcn_perm(t3, t2, 0x05040100u);
  o3 = __builtin_amdgcn_perm(t3, t2, 0x07060302u);
}

__device__ __forceinline__ int block_pair(int b1, int b2, int nb) {
  // index of (b1 <= b2) in row-major upper-triangle order of nb blocks
  return b1 * nb - b1 * (b1 - 1) / 2 + (b2 - b1);
}

template <int NB, int CW, int CPW, int IPW, int NST>
struct MfmaCfg {
  static constexpr int NBP = NB * (NB + 1) / 2;        // 16x16 block pairs
  static constexpr int WIDTH = CW;                     // channels of a tile
  static constexpr int KEY = ((NB * 128 + CW) * 16 + CPW) * 128 + IPW * 8 + NST;
  static constexpr int NWAVE = CW / CPW;
  static constexpr int NTHR = 64 * NWAVE;
  static constexpr int SEGS = CW / 16;                 // 16-byte units per row
  static constexpr int UPB = TC * SEGS;                // units per beam per chunk
  static constexpr int STAGE = IPW * NWAVE * 1024;     // bytes per chunk buffer
  static constexpr int NGRP = CPW >= 4 ? CPW / 4 : 1;  // dword groups of 4 channels
  // LDS: the ring of NST chunk buffers. After the last chunk the same space
  // holds the epilogue's offset sums [MAXB][CW] and its staging rows.
  static constexpr int MAXB = 16 * NB - 1;             // beams (plus the ones row)
  static constexpr int MAXROW = MAXB + MAXB * (MAXB + 1) / 2;
  static constexpr int LDS_MAX = 160 * 1024;
  static constexpr int RING = NST * STAGE;
  static constexpr int SXL_OFF = 0;
  static constexpr int STG_OFF = SXL_OFF + MAXB * CW * 4;
  // worst case of the staging: one wave's channels per pass at the largest
  // beam count
  static constexpr int STG_MIN = MAXROW * (CPW + 1) * 4;
  // the workgroup's LDS: the ring, or the epilogue's minimum if larger (more
  // epilogue passes in less space), 1 KB granules. A tile whose ring is at
  // most half the CU's LDS leaves room for a second workgroup, whose loads
  // then stream during this one's epilogue.
  static constexpr int NEED = RING > STG_OFF + STG_MIN ? RING : STG_OFF + STG_MIN;
  static constexpr int LDS = (NEED + 1023) / 1024 * 1024 < LDS_MAX
                                 ? (NEED + 1023) / 1024 * 1024
                                 : LDS_MAX;
  static constexpr int STG_BYTES = LDS - STG_OFF;
  static constexpr int SLOTS = 256 * (LDS_MAX / LDS < 2 ? 1 : 2);  // workgroups the chip holds
  static constexpr bool DIRECT = false;                // records staged in LDS
  static constexpr bool FITS = RING <= LDS_MAX && STG_BYTES >= STG_MIN;
};

// LDS unit (16 bytes) of (beam, row, segment) inside a chunk buffer
template <int UPB, int SEGS>
__device__ __forceinline__ int unit_of(int beam, int row, int seg) {
  const int lin = beam * UPB + row * SEGS + seg;
  return lin ^ ((beam + 2 * (row >> 3)) & 7);
}

// wait until at most N vector-memory operations of this wave are in flight,
// then meet the workgroup; the memory clobber keeps LDS accesses on their side
template <int N>
__device__ __forceinline__ void vm_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int IPW, int NST>
__device__ __forceinline__ void wait_chunk(int ahead) {
  // 'ahead' chunks (IPW loads each) were requested after the one about to be
  // consumed; at most NST - 1
  if constexpr (NST >= 4) {
    if (ahead >= 3) { vm_wait_barrier<3 * IPW>(); return; }
  }
  if constexpr (NST >= 3) {
    if (ahead >= 2) { vm_wait_barrier<2 * IPW>(); return; }
  }
  if (ahead >= 1) { vm_wait_barrier<IPW>(); return; }
  vm_wait_barrier<0>();
}

// Tiles per XCD group: 1 KB of contiguous row bytes by default (measured best
// for the 4 KB-row FAST layout); a tune entry may choose another size. n: the
// workgroups they are dealt to. A launch of fewer than 8 G workgroups gets eight
// groups of what it has: ungrouped, the tiles that share a 128-byte line are fetched
// through all eight L2s (79 beams x 256 channels x 203450 samples, 256 workgroups of
// 16 channels: 4643 us, grouped 2073).
__host__ __device__ inline int group_tiles(int G, int64_t n) {
  return (int64_t)8 * G > n ? (int)(n / 8) : G;
}
int group_tiles(int cw, int group_bytes_override, int64_t n) {
  const int gb = group_bytes_override > 0 ? group_bytes_override : 1024;
  return group_tiles(gb / cw, n);
}

// workgroup -> tile: G consecutive channel tiles of a sub-interval (G CW
// contiguous bytes of every row) go to G workgroups that are dispatched
// back to back on the same XCD (workgroup ids w, w + 8, w + 16, ...): the
// hardware dispatcher then keeps adjacent tiles in step, and each row is
// fetched in long runs through one L2
__device__ __forceinline__ int xcd_group(int w, int n, int G) {
  const int full = G > 1 ? (n / (8 * G)) * (8 * G) : 0;
  if (w >= full) return w;
  const int u = w / (8 * G), rem = w % (8 * G);
  return G * (8 * u + rem % 8) + rem / 8;
}

// Workgroup w's share of a launch of ntiles tiles: tiles below nwhole go to one
// workgroup each, the samples of the later ones are shared out to `parts`.
// Sub-interval k, channel tile ct, samples [r0, r0 + n) of its L (whole chunks
// of TC; n <= 0: more parts than this needs). A workgroup of parts > 1 adds its
// sums to the outputs (zero before the launch, or the caller's). G: the group of
// the whole tiles in the low half, of the shared ones in the high half.
struct Tile {
  int k, ct, part, parts, r0, n;
};
__device__ __forceinline__ Tile tile_of(int w, int ntiles, int nct, int nwhole, int parts, int G,
                                        int ksplit, int L, int Llast) {
  Tile t;
  int tile;
  if (w < nwhole) {
    tile = xcd_group(w, nwhole, G & 0xffff);
    t.part = 0;
    t.parts = 1;
  } else {
    const int tail = ntiles - nwhole;
    const int m = xcd_group(w - nwhole, tail * parts, G >> 16);
    tile = nwhole + m % tail;
    t.part = m / tail;
    t.parts = parts;
  }
  t.k = tile / nct;
  t.ct = tile % nct;
  const int Lk = t.k % ksplit == ksplit - 1 ? Llast : L;
  const int per = ((Lk + TC - 1) / TC + t.parts - 1) / t.parts * TC;
  t.r0 = t.part * per;
  t.n = Lk - t.r0 < per ? Lk - t.r0 : per;
  return t;
}

// Second half of an epilogue, one pass over cwp of a tile's channels from its
// channel h cwp on: the staged offset sums of the pairs (rows of cwp + 1 at stg,
// the pad keeps the scattered writes of one instruction in distinct banks) and
// the S'_a at sxl become raw sums
//     S_a = S'_a + 128 L,   S_ab = S'_ab + 128 (S'_a + S'_b) + 16384 L
// in coalesced runs. Rows layout: thread t stores channel t mod cwp of rows t / cwp, t / cwp
// + rstep, ... (runs of consecutive cells); cell records: thread t stores rows
// t mod rstep, + rstep, ... of channel t / rstep (runs of consecutive rows).
__device__ __forceinline__ void store_sums(const int32_t* stg, const int32_t* sxl, int nbeam, int cw,
                                           int cwp, int h, int c0, int nchan, int64_t k,
                                           int64_t ncell, int layout, int32_t* __restrict__ sum_x,
                                           int32_t* __restrict__ sum_xy, uint32_t cnt, bool shared,
                                           int accumulate, int tid, int nthr) {
  const int rstep = nthr / cwp;
  const int ch = layout ? tid / rstep : tid % cwp;
  const int row0 = layout ? tid % rstep : tid / cwp;
  const int chl = h * cwp + ch;
  const int chan = c0 + chl;
  if (chan >= nchan) return;
  const int np = nbeam * (nbeam + 1) / 2;
  const int64_t cell = k * nchan + chan;
  int32_t* dx = layout ? sum_x + cell * (nbeam + np) : sum_x + cell;
  int32_t* dxy = layout ? dx + nbeam : sum_xy + cell;
  const int64_t ld = layout ? 1 : ncell;
  auto put = [&](int32_t* dst, uint32_t raw) {
    if (shared) atomicAdd((unsigned*)dst, raw);   // integers: exact in any order
    else *dst = accumulate ? (int32_t)((uint32_t)*dst + raw) : (int32_t)raw;
  };
  const int32_t* sx = sxl + chl;
  for (int a = row0; a < nbeam; a += rstep) put(dx + a * ld, (uint32_t)sx[a * cw] + 128u * cnt);
  int a = 0, b = row0;
  for (int q = row0; q < np; q += rstep, b += rstep) {
    while (b >= nbeam) { ++a; b -= nbeam - a; }   // pair q is (a, b)
    put(dxy + q * ld, (uint32_t)stg[q * (cwp + 1) + ch] +
                          128u * ((uint32_t)sx[a * cw] + (uint32_t)sx[b * cw]) + 16384u * cnt);
  }
}

template <int NB, int CW, int CPW, int IPW, int NST>
__global__ __launch_bounds__((MfmaCfg<NB, CW, CPW, IPW, NST>::NTHR), 1) void ccm_mfma_kernel(
    BeamPtrs bp, int nbeam, int nchan, int64_t row_stride, int64_t t0, int L, int nsub,
    int nct, int32_t* __restrict__ sum_x, int32_t* __restrict__ sum_xy,
    int32_t* __restrict__ count, int accumulate, int G, int nh, int layout,
    int64_t kstride, int ksplit, int Llast, int nwhole, int parts, const CcmItem* __restrict__ items, int nitem) {
  using C = MfmaCfg<NB, CW, CPW, IPW, NST>;
  // the beam pointer table is the first kernel argument: index it in place
  const uint8_t* const* beam_tab = (const uint8_t* const*)__builtin_amdgcn_kernarg_segment_ptr();
  int w = blockIdx.x;
  if (items) {
    // batched launch: workgroups [wg0, wg0 + 8 ceil(tiles / 8)) belong to one
    // block (its own shape, beams, sub-intervals and sum buffers); find it
    int lo = 0, hi = nitem - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (items[mid].wg0 <= w) lo = mid; else hi = mid - 1;
    }
    const CcmItem& it = items[lo];
    beam_tab = it.beams;
    nbeam = it.nbeam;
    nchan = it.nchan;
    row_stride = it.row_stride;
    t0 = it.t0;
    L = it.L;
    nsub = it.nsub;
    nct = it.nct;
    nh = it.nh;
    sum_x = it.sum_x;
    sum_xy = it.sum_xy;
    count = it.count;
    layout = it.layout;
    parts = it.parts;
    w -= it.wg0;
    if (w >= nsub * nct * parts) return;      // padding to a multiple of 8 workgroups
    nwhole = 0;
    G = group_tiles(G, nsub * nct * parts) << 16;
    kstride = 0;
    ksplit = 1;
    Llast = L;
  }
  // sub-interval k of the launch starts at t0 + (k / ksplit) kstride +
  // (k mod ksplit) L: with ksplit = 1 and kstride = L they are back to back; a
  // longer stride sums one time chunk of each of several long sub-intervals,
  // and ksplit > 1 cuts each of those into ksplit consecutive chunks of L, the
  // last one of Llast <= L
  if (kstride == 0) kstride = L;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  // epilogue areas, over the drained ring
  int32_t* sxl = (int32_t*)(lds + C::SXL_OFF);       // [nbeam][CW] offset sums S'_a
  int32_t* stg = (int32_t*)(lds + C::STG_OFF);       // [npair][CW / nh + 1] output staging
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t ncell = (int64_t)nsub * nchan;
  const Tile tl = tile_of(w, nsub * nct, nct, nwhole, parts, G, ksplit, L, Llast);
  const int k = tl.k, r0 = tl.r0, Lp = tl.n, c0 = tl.ct * CW;
  if (Lp <= 0) return;
  const int nchunk = (Lp + TC - 1) / TC;

  // Per chunk this thread's lane fills unit (64 q + lane) of the buffer for
  // q = wave + NWAVE i, i < IPW; decode which (beam, row, seg) lands there.
  // Units past the beams, rows past the sub-interval and segments past the
  // row read a valid dummy address (never consumed), so every wave issues
  // exactly IPW loads per chunk and vmcnt counts stay uniform.
  const uint8_t* src_base[IPW];
  int src_row[IPW], src_col[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int s = 64 * (wave + C::NWAVE * i) + lane;
    const int hi = s & ~7;
    const int bh = hi / C::UPB, rh = (hi % C::UPB) / C::SEGS;
    const int lin = s ^ ((bh + 2 * (rh >> 3)) & 7);
    const int b = lin / C::UPB, r = (lin % C::UPB) / C::SEGS, g = lin % C::SEGS;
    src_base[i] = beam_tab[b < nbeam ? b : 0];
    src_row[i] = b < nbeam ? r : -1;
    src_col[i] = 16 * g;
  }
  // DMA of chunk `chunk` into ring buffer `slot`
  auto issue = [&](int chunk, int slot) {
    uint8_t* buf = lds + slot * C::STAGE;
    const int rows = min(TC, Lp - chunk * TC);
    const int64_t row = t0 + (int64_t)(k / ksplit) * kstride + (int64_t)(k % ksplit) * L + r0 +
                        (int64_t)chunk * TC;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int64_t col = c0 + src_col[i];
      const bool ok = src_row[i] >= 0 && col < row_stride;
      const int r = (ok && src_row[i] < rows) ? src_row[i] : 0;
      const uint8_t* src = src_base[i] + (row + r) * row_stride + (ok ? col : 0);
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)src,
          (__attribute__((address_space(3))) void*)(buf + 1024 * (wave + C::NWAVE * i)), 16, 0, 0);
    }
  };

  v4i acc[CPW][C::NBP];
  auto zero_acc = [&]() {
#pragma unroll
    for (int c = 0; c < CPW; ++c)
#pragma unroll
      for (int p = 0; p < C::NBP; ++p) acc[c][p] = v4i{0, 0, 0, 0};
  };
  zero_acc();

  const int li = lane & 15;     // row (beam) within a 16-row block
  const int kg = lane >> 4;     // which 8 of the chunk's 32 rows this lane supplies
  const int cb = wave * CPW;    // first channel of this wave within the tile

  auto compute_chunk = [&](int slot) {
    const uint8_t* src = lds + slot * C::STAGE;
#pragma unroll
    for (int grp = 0; grp < C::NGRP; ++grp) {
      const int ch4 = (CPW >= 4) ? (cb + 4 * grp) : (cb & ~3);
      const int seg = ch4 >> 4, wrd = (ch4 & 15) >> 2;
      long op[NB][4];
#pragma unroll
      for (int bb = 0; bb < NB; ++bb) {
        const int beam = 16 * bb + li;
        uint32_t r[8];
        if (beam < nbeam) {
          // rows 8 kg + j: the swizzle only permutes units within aligned
          // groups of 8, so unit(j) = unit(j mod P) + 8 (j / P), P = 8 / SEGS,
          // and the 8 reads need P base addresses plus immediate offsets
          constexpr int P = 8 / C::SEGS;
          const uint8_t* basep[P];
#pragma unroll
          for (int m = 0; m < P; ++m)
            basep[m] = src + 16 * unit_of<C::UPB, C::SEGS>(beam, 8 * kg + m, seg) + 4 * wrd;
#pragma unroll
          for (int j = 0; j < 8; ++j)
            r[j] = *(const uint32_t*)(basep[j % P] + 128 * (j / P)) ^ OFFSET_XOR;
        } else {
          const uint32_t v = (beam == nbeam) ? 0x01010101u : 0u;
#pragma unroll
          for (int j = 0; j < 8; ++j) r[j] = v;
        }
        uint32_t o[8];
        transpose4x4(r[0], r[1], r[2], r[3], o[0], o[1], o[2], o[3]);
        transpose4x4(r[4], r[5], r[6], r[7], o[4], o[5], o[6], o[7]);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          op[bb][c] = (long)(((uint64_t)o[4 + c] << 32) | (uint64_t)o[c]);
      }
      if constexpr (CPW >= 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int slot = 4 * grp + c;
#pragma unroll
          for (int b1 = 0; b1 < NB; ++b1)
#pragma unroll
            for (int b2 = b1; b2 < NB; ++b2) {
              const int p = block_pair(b1, b2, NB);
              acc[slot][p] = __builtin_amdgcn_mfma_i32_16x16x32_i8(op[b1][c], op[b2][c],
                                                                   acc[slot][p], 0, 0, 0);
            }
        }
      } else {
        // this wave owns channels (cb & 3) .. (cb & 3) + CPW - 1 of the dword
        const int coff = cb & 3;
#pragma unroll
        for (int slot = 0; slot < CPW; ++slot) {
          const int c = coff + slot;                 // wave-uniform
          long sel[NB];
#pragma unroll
          for (int bb = 0; bb < NB; ++bb)
            sel[bb] = c == 0 ? op[bb][0] : c == 1 ? op[bb][1] : c == 2 ? op[bb][2] : op[bb][3];
#pragma unroll
          for (int b1 = 0; b1 < NB; ++b1)
#pragma unroll
            for (int b2 = b1; b2 < NB; ++b2) {
              const int p = block_pair(b1, b2, NB);
              acc[slot][p] = __builtin_amdgcn_mfma_i32_16x16x32_i8(sel[b1], sel[b2],
                                                                   acc[slot][p], 0, 0, 0);
            }
        }
      }
    }
  };

  // Epilogue. The offset sums S'_a (ones column) go to LDS first. Then, in nh
  // passes over the tile's channels (whole waves per pass), the waves of the
  // pass write their raw offset sums of the pairs to the staging rows, and the
  // whole workgroup converts and stores them. It runs over the drained ring;
  // its barriers wait for LDS only.
  auto lds_barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  const int cwp = CW / nh;
  auto epilogue = [&]() {
    const int jn = nbeam & 15, bn = nbeam >> 4;
    if (li == jn) {
#pragma unroll
      for (int c = 0; c < CPW; ++c)
#pragma unroll
        for (int b1 = 0; b1 < NB; ++b1)
#pragma unroll
          for (int b2 = b1; b2 < NB; ++b2) {
            if (b2 != bn) continue;
            const int p = block_pair(b1, b2, NB);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int a = 16 * b1 + 4 * kg + r;
              if (a < nbeam) sxl[a * CW + cb + c] = acc[c][p][r];
            }
          }
    }
    const int mypass = cb / cwp;
    for (int h = 0; h < nh; ++h) {
      if (mypass == h) {
#pragma unroll
        for (int b1 = 0; b1 < NB; ++b1)
#pragma unroll
          for (int b2 = b1; b2 < NB; ++b2) {
            const int p = block_pair(b1, b2, NB);
            const int b = 16 * b2 + li;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int a = 16 * b1 + 4 * kg + r;
              if (a <= b && b < nbeam) {
                const int row = a * nbeam - a * (a - 1) / 2 + (b - a);
                int32_t* dst = stg + row * (cwp + 1) + (cb - h * cwp);
#pragma unroll
                for (int c = 0; c < CPW; ++c) dst[c] = acc[c][p][r];
              }
            }
          }
      }
      lds_barrier();
      store_sums(stg, sxl, nbeam, CW, cwp, h, c0, nchan, k, ncell, layout, sum_x,
                 sum_xy, (uint32_t)Lp, tl.parts > 1, accumulate, tid, C::NTHR);
      lds_barrier();
    }
    if (c0 == 0 && tl.part == 0 && tid == 0) {
      const int Lk = k % ksplit == ksplit - 1 ? Llast : L;
      count[k] = accumulate ? count[k] + Lk : Lk;
    }
  };

  // ring of NST buffers: chunks c+1 .. c+NST-2 (and c+NST-1 once issued) are
  // in flight while chunk c is consumed
  for (int c = 0; c < NST - 1 && c < nchunk; ++c) issue(c, c);
  for (int c = 0; c < nchunk; ++c) {
    const int last_issued = min(c + NST - 2, nchunk - 1);
    const int slot = c % NST;
    wait_chunk<IPW, NST>(last_issued - c);          // chunk c complete in LDS
    if (c + NST - 1 < nchunk) issue(c + NST - 1, (c + NST - 1) % NST);  // buffer of c - 1
    if (c == nchunk - 1 && Lp % TC != 0) {
      // short last chunk: its rows past the range hold dummy data; overwrite
      // them with 0x80 bytes (0 after the offset XOR)
      const int rows = Lp - c * TC;
      uint8_t* buf = lds + slot * C::STAGE;
      const int nu = nbeam * (TC - rows) * C::SEGS;
      for (int u = tid; u < nu; u += C::NTHR) {
        const int b = u / ((TC - rows) * C::SEGS);
        const int rr = rows + (u / C::SEGS) % (TC - rows);
        const int sg = u % C::SEGS;
        *(uint4*)(buf + 16 * unit_of<C::UPB, C::SEGS>(b, rr, sg)) =
            make_uint4(OFFSET_XOR, OFFSET_XOR, OFFSET_XOR, OFFSET_XOR);
      }
      lds_barrier();
    }
    compute_chunk(slot);
  }
  // every wave is past its last read of the ring before the epilogue reuses it
  lds_barrier();
  epilogue();
}

// Packed engine (16 NBF beams and up to 8 more, NBF = 1..4): wider rows for the
// same registers. Narrow pieces of a row cost the memory system almost as much as
// whole 128-byte lines (bare loads, one workgroup per CU: pieces of 16 / 32 / 64 /
// 128 bytes 2.3 / 3.6 / 5.8 / 6.4 TB/s), so the tile should be as wide as the
// accumulators allow, and these are mostly padding to 16-row blocks. Here only
// the NBF full blocks are held per channel; the nbeam - 16 NBF beams left of Q
// channels share one operand P of 16 rows, RQ = 16 / Q to a channel: lane li holds
// beam 16 NBF + li % RQ of channel li / RQ:
//     full x left    X_b P_c^T, P_c = P with the other channels' lanes zero: the
//                    Q channels land in disjoint columns of one accumulator;
//     left x left    P P^T, of which the diagonal blocks are the Q channels'
//                    (the rest mixes channels and is not read);
// The offset sums S'_a come out of the same products where an operand has a row
// to spare for ones (nbeam % 16 < 8); for 8 beams left they have accumulators of
// their own, X_b E_j with E_j all ones in column j and zero elsewhere, the S'_a
// of 16 operands to one. Accumulator registers per 4 channels: 19 beams 24 instead
// of 48, 36 beams 72 instead of 96, 72 beams 208 instead of 240.
//
// That gives 32..40 beams tiles of 64 channels instead of 32 and 48..72 beams 32
// instead of 16; 16..19 beams keep 64 on half the waves, so that a second
// workgroup of the CU loads during the epilogue. The ring holds stages of 16 rows
// (half a K = 32 step, the first half's operands wait in registers): a wider stage
// leaves as many bytes in flight. Records of 48 beams and more go to memory
// straight from the accumulators: staging them in LDS was a quarter of the launch
// (36 beams measured better staged, 425 against 450 us). Bound: the memory system
// at the piece size, then the epilogue. Whole blocks -> packed: 36 beams x 1000
// channels x 1024 samples x 39 585 -> 425 us (3.4 TB/s); 19 x 4096 x 2048 x 99 3241
// -> 3130 us (5.0 TB/s), x 1024 x 1017 x 60 277 -> 254 us; 72 x 1024 x 512 x 40 as
// cell records 1019 -> 697 us, rows 1179 -> 980.
// The instances of 64 beams and more overflow their 256 registers: 48 bytes of
// scratch a lane up to 67 beams, 136 from 68 on, where one accumulator is stored and
// reloaded in every K = 32 step. The reload waits for the loads of all stages ahead,
// so the ring is empty when a step ends: 2.2 TB/s at 72 beams where bare 32-byte
// pieces reach 3.6. (The extra operations make the counted waits wait longer, never
// shorter.)
//
// A wave owns CPW channels and reads a row's CPW bytes of a beam in one LDS load;
// 16-byte units are XOR-swizzled by the beam, which spreads the 16 beams of a
// load over all banks. Load addresses are recomputed per stage from the beam
// table (scalar loads), which leaves their registers to the accumulators.
template <int NBF, int Q, bool ONES>
struct PackCfg {
  static constexpr int TR = 16;                        // rows per stage
  static constexpr int CW = NBF <= 2 ? 64 : 32;
  static constexpr int WIDTH = CW;
  static constexpr int KEY = (1 << 28) + (NBF * 8 + Q) * 2 + ONES;
  static constexpr int NWAVE = NBF == 2 ? 16 : 8;      // as the accumulators allow
  static constexpr bool DIRECT = NBF >= 3;             // records straight from registers
  static constexpr bool PAIR = NBF == 1;               // both stages of a step land before it
  static constexpr int NTHR = 64 * NWAVE;
  static constexpr int CPW = CW / NWAVE;
  static constexpr int NG = CPW / 4;                   // groups of 4 channels per wave
  static constexpr int SEGS = CW / 16;
  static constexpr int UPB = TR * SEGS;                // 16-byte units per beam per stage
  static constexpr int RQ = 16 / Q;                    // rows of a packed operand per channel
  static constexpr int PG = 4 / Q;                     // packed operands per group
  static constexpr int NP = NBF * (NBF + 1) / 2;       // pairs of full blocks
  // where the accumulators leave few registers, the second half's operands are
  // read and used two channels of a group at a time
  static constexpr bool HALVES = NBF == 4 || (NBF <= 2 && !ONES);
  // offset sums without the ones row: SG channels' full-block columns and their
  // packed operands' per accumulator
  static constexpr int SG = NBF == 1 ? 8 : NBF <= 3 ? 4 : 2;
  static constexpr int NS = ONES ? 0 : CPW / SG;
  static constexpr int MAXB = 16 * NBF + RQ - ONES;
  // loads of 1 KB per stage: ceil(nbeam SEGS / 4), LO or LO + 1 to a wave
  static constexpr int LO = NBF <= 2 ? 2 : NBF;
  static constexpr int LDS_MAX = (NBF == 1 ? 80 : 160) * 1024;   // two workgroups per CU, or one
  static constexpr int STAGE = (MAXB * SEGS + 3) / 4 * 1024;
  static constexpr int NST = LDS_MAX / STAGE < 4 ? LDS_MAX / STAGE : 4;
  static constexpr int SXS = CW + 1;                   // row stride of the offset sums
  static constexpr int STG_OFF = (MAXB * SXS * 4 + 15) / 16 * 16;
  static constexpr int LDS = LDS_MAX;
  static constexpr int STG_BYTES = LDS - STG_OFF;
  static constexpr int SLOTS = NBF == 1 ? 512 : 256;
  static_assert(NST >= 3 && STAGE <= (LO + 1) * NWAVE * 1024, "stage");
  static_assert(STG_BYTES >= MAXB * (MAXB + 1) / 2 * (CPW + 1) * 4, "staging");
  static_assert(ONES || NBF * SG + SG / Q <= 16, "offset sum columns");
  // epilogue passes for nbeam beams (whole waves each)
  static int passes(int nbeam) {
    const int np = nbeam * (nbeam + 1) / 2;
    int nh = 1;
    while (nh < NWAVE && np * (CW / nh + 1) * 4 > STG_BYTES) nh *= 2;
    return nh;
  }
};

// Wait until stage h has landed, `ahead` later ones of LD loads each being under
// way, and meet the workgroup. This wave's LDS reads have returned too: the
// buffer they read is refilled after the barrier.
template <int LD, int NST>
__device__ __forceinline__ void wait_stage(int ahead) {
  if constexpr (NST >= 4) {
    if (ahead >= 2) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * LD) : "memory");
      return;
    }
  }
  if (ahead >= 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LD) : "memory");
  else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

template <int NBF, int Q, bool ONES>
__global__ __launch_bounds__((PackCfg<NBF, Q, ONES>::NTHR), NBF <= 2 ? 4 : 2) void ccm_pack_kernel(
    BeamPtrs bp, int nbeam, int nchan, int64_t row_stride, int64_t t0, int L, int nsub,
    int nct, int32_t* __restrict__ sum_x, int32_t* __restrict__ sum_xy,
    int32_t* __restrict__ count, int accumulate, int G, int nh, int layout, int64_t kstride,
    int ksplit, int Llast, int nwhole, int parts, const CcmItem* __restrict__ items, int nitem) {
  using C = PackCfg<NBF, Q, ONES>;
  constexpr int CW = C::CW, CPW = C::CPW, TR = C::TR, SEGS = C::SEGS, UPB = C::UPB, NST = C::NST;
  constexpr int RQ = C::RQ, PG = C::PG, NG = C::NG, SG = C::SG, NS = C::NS, SXS = C::SXS;
  constexpr int AHEAD = C::PAIR ? NST - 2 : NST - 1;   // stages under way during the products
  // the beam table in constant memory: the first kernel argument or the item's
  using Tab = const uint64_t __attribute__((address_space(4)))*;
  Tab beams = (Tab)__builtin_amdgcn_kernarg_segment_ptr();
  int w = blockIdx.x;
  if (items) {
    int lo = 0, hi = nitem - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (items[mid].wg0 <= w) lo = mid; else hi = mid - 1;
    }
    const CcmItem& it = items[lo];
    beams = (Tab)(uintptr_t)it.beams;
    nbeam = it.nbeam;
    nchan = it.nchan;
    row_stride = it.row_stride;
    t0 = it.t0;
    L = it.L;
    nsub = it.nsub;
    nct = it.nct;
    nh = it.nh;
    sum_x = it.sum_x;
    sum_xy = it.sum_xy;
    count = it.count;
    layout = it.layout;
    parts = it.parts;
    w -= it.wg0;
    if (w >= nsub * nct * parts) return;      // padding to a multiple of 8 workgroups
    nwhole = 0;
    G = group_tiles(G, nsub * nct * parts) << 16;
    kstride = 0;
    ksplit = 1;
    Llast = L;
  }
  if (kstride == 0) kstride = L;
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  int32_t* sxl = (int32_t*)lds;                      // epilogue areas, over the drained ring
  int32_t* stg = (int32_t*)(lds + C::STG_OFF);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ncell = (int64_t)nsub * nchan;
  const Tile tl = tile_of(w, nsub * nct, nct, nwhole, parts, G, ksplit, L, Llast);
  const int k = tl.k, Lp = tl.n, c0 = tl.ct * CW;
  if (Lp <= 0) return;
  const int stage = (nbeam * SEGS + 3) / 4 * 1024;         // bytes of a ring buffer
  const int nstage = (Lp + 2 * TR - 1) / (2 * TR) * 2;   // whole K = 32 steps
  const int64_t row0 = t0 + (int64_t)(k / ksplit) * kstride + (int64_t)(k % ksplit) * L + tl.r0;

  // DMA of stage j into ring buffer `slot`: lane l of load q = wave + NWAVE i < nld
  // fills unit s = 64 q + l, which holds unit s ^ (beam mod 16) of the stage in
  // (beam, row, segment) order. Beams, rows and segments past the end read a
  // valid address instead (never consumed).
  const int nld = (nbeam * SEGS + 3) / 4;
  const bool more = wave + C::NWAVE * C::LO < nld;   // LO + 1 loads, else LO
  const bool near_rows = row_stride < (1 << 27);
  // beam and unit of lane l in load q
  auto unit_at = [&](int q, int l, int* b, int* u) {
    if constexpr (SEGS >= 4) {
      *b = 64 * q / UPB;
      *u = (64 * q % UPB + l) ^ (*b & 15);
    } else {
      *b = 2 * q + (l >> 5);
      *u = (l & 31) ^ (*b & 15);
    }
  };
  auto base_of = [&](int q, int l) {
    if constexpr (SEGS >= 4) {
      return beams[min(64 * q / UPB, nbeam - 1)];
    } else {
      const uint64_t b0 = beams[min(2 * q, nbeam - 1)], b1 = beams[min(2 * q + 1, nbeam - 1)];
      return l < 32 ? b0 : b1;
    }
  };
  auto offset_of = [&](int q, int l) {                 // of a whole stage's lanes
    int b, u;
    unit_at(q, l, &b, &u);
    const int col = c0 + 16 * (u % SEGS);
    return (b < nbeam) & (col < row_stride) ? (uint32_t)(u / SEGS) * (uint32_t)row_stride + col
                                            : 0u;
  };
  uint32_t off[C::LO + 1];
#pragma unroll
  for (int i = 0; i <= C::LO; ++i) off[i] = C::HALVES ? 0 : offset_of(wave + C::NWAVE * i, lane);
  auto issue = [&](int j, int slot) {
    uint8_t* buf = lds + slot * stage;
    const int rows = Lp - j * TR;                      // <= 0: all past the end
    const int64_t at = (row0 + (rows > 0 ? j * TR : 0)) * row_stride;
    int l = lane;
    asm volatile("" : "+v"(l));              // recomputed here, not kept over the loop
    auto load = [&](int q, const uint8_t* src) {
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)src,
          (__attribute__((address_space(3))) void*)(buf + 1024 * q), 16, 0, 0);
    };
    if (rows >= TR && near_rows) {
#pragma unroll
      for (int i = 0; i <= C::LO; ++i) {
        const int q = wave + C::NWAVE * i;
        if (i < C::LO || more)
          load(q, (const uint8_t*)(base_of(q, l) + at) + (C::HALVES ? offset_of(q, l) : off[i]));
      }
    } else {
#pragma unroll 1
      for (int i = 0; i < C::LO + more; ++i) {
        const int q = wave + C::NWAVE * i;
        int b, u;
        unit_at(q, l, &b, &u);
        const int col = c0 + 16 * (u % SEGS);
        const bool ok = (b < nbeam) & (col < row_stride);
        const int r = ok & (u / SEGS < rows) ? u / SEGS : 0;
        load(q, (const uint8_t*)(base_of(q, l) + at) + (int64_t)r * row_stride + (ok ? col : 0));
      }
    }
  };

  v4i acc[CPW][C::NP], accp[NG * PG][NBF], accr[NG * PG], accs[NS + 1];
#pragma unroll
  for (int c = 0; c < CPW; ++c)
#pragma unroll
    for (int p = 0; p < C::NP; ++p) acc[c][p] = v4i{0, 0, 0, 0};
#pragma unroll
  for (int g = 0; g < NG * PG; ++g) {
    accr[g] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < NBF; ++b) accp[g][b] = v4i{0, 0, 0, 0};
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) accs[i] = v4i{0, 0, 0, 0};

  const int li = lane & 15;     // row (beam) within a 16-row block
  const int kg = lane >> 4;     // which 4 of a stage's 16 rows this lane supplies
  const int cb = wave * CPW;    // first channel of this wave within the tile
  const int cs = li / RQ;       // this lane's channel of a packed operand

  // operands of one stage: o[group][block][channel] and p[group][packed], four
  // samples each; of channels [lo, lo + 2) of each group, or of all four
  auto read_stage = [&](int slot, auto lo_c, auto nc_c, uint32_t (&o)[NG][NBF][4],
                        uint32_t (&p)[NG][PG]) {
    constexpr int lo = lo_c, nc = nc_c;
    const uint8_t* src = lds + slot * stage;
    int l = lane;
    if constexpr (C::HALVES) asm volatile("" : "+v"(l));   // addresses not kept either
    const int li = l & 15, kg = l >> 4;
    const uint32_t psel = (uint32_t)(li / RQ) * 0x0101u + 0x0400u;
#pragma unroll
    for (int bb = 0; bb <= NBF; ++bb) {
      const int beam = bb < NBF ? 16 * bb + li : min(16 * NBF + li % RQ, nbeam - 1);
      uint32_t r[4][NG];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int unit = (beam * UPB + (4 * kg + j) * SEGS + (cb >> 4)) ^ (beam & 15);
        const uint8_t* a = src + 16 * unit + (cb & 15);
        if constexpr (NG == 4) {
          const uint4 v = *(const uint4*)a;
          r[j][0] = v.x; r[j][1] = v.y; r[j][2] = v.z; r[j][3] = v.w;
        } else if constexpr (NG == 2) {
          const uint2 v = *(const uint2*)a;
          r[j][0] = v.x; r[j][1] = v.y;
        } else {
          r[j][0] = *(const uint32_t*)a;
        }
      }
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (bb < NBF) {
          uint32_t t[4];
          transpose4x4(r[0][g], r[1][g], r[2][g], r[3][g], t[0], t[1], t[2], t[3]);
#pragma unroll
          for (int c = lo; c < lo + nc; ++c) o[g][bb][c] = t[c] ^ OFFSET_XOR;
        } else {
#pragma unroll
          for (int q = lo / Q; q < (lo + nc + Q - 1) / Q; ++q) {
            const uint32_t s = psel + 0x0101u * (uint32_t)(q * Q);
            const uint32_t t0 = __builtin_amdgcn_perm(r[1][g], r[0][g], s);
            const uint32_t t1 = __builtin_amdgcn_perm(r[3][g], r[2][g], s);
            p[g][q] = __builtin_amdgcn_perm(t1, t0, 0x05040100u) ^ OFFSET_XOR;
            if (ONES && 16 * NBF + li % RQ == nbeam) p[g][q] = 0x01010101u;
          }
        }
      }
      if constexpr (NBF == 4) asm volatile("" ::: "memory");   // one block's rows at a time
    }
  };
  auto mfma = [](long a, long b, v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x32_i8(a, b, c, 0, 0, 0);
  };
  auto join = [](uint32_t lo, uint32_t hi) { return (long)(((uint64_t)hi << 32) | lo); };
  auto multiply = [&](auto lo_c, auto nc_c, const uint32_t (&ol)[NG][NBF][4],
                      const uint32_t (&oh)[NG][NBF][4], const uint32_t (&pl)[NG][PG], const uint32_t (&ph)[NG][PG]) {
    constexpr int lo = lo_c, nc = nc_c;
    int l = lane;
    if constexpr (C::HALVES) asm volatile("" : "+v"(l));
    const int li = l & 15, cs = li / RQ;
    auto ones = [&](int col) {
      const uint32_t v = li == col ? 0x01010101u : 0u;
      return (long)(((uint64_t)v << 32) | v);
    };
#pragma unroll
    for (int g = 0; g < NG; ++g) {
#pragma unroll
      for (int c = lo; c < lo + nc; ++c) {
        const int ch = 4 * g + c, q = c / Q;
        long x[NBF];
#pragma unroll
        for (int b = 0; b < NBF; ++b) x[b] = join(ol[g][b][c], oh[g][b][c]);
        const bool mine = cs == c % Q;
        const long pc = join(mine ? pl[g][q] : 0u, mine ? ph[g][q] : 0u);
#pragma unroll
        for (int b1 = 0; b1 < NBF; ++b1) {
#pragma unroll
          for (int b2 = b1; b2 < NBF; ++b2)
            acc[ch][block_pair(b1, b2, NBF)] =
                mfma(x[b1], x[b2], acc[ch][block_pair(b1, b2, NBF)]);
          accp[g * PG + q][b1] = mfma(x[b1], pc, accp[g * PG + q][b1]);
          if constexpr (!ONES)
            accs[ch / SG] = mfma(x[b1], ones(b1 * SG + ch % SG), accs[ch / SG]);
        }
      }
#pragma unroll
      for (int q = (lo + Q - 1) / Q; q < (lo + nc + Q - 1) / Q; ++q) {
        const int ch = 4 * g + q * Q;
        const long x = join(pl[g][q], ph[g][q]);
        accr[g * PG + q] = mfma(x, x, accr[g * PG + q]);
        if constexpr (!ONES)
          accs[ch / SG] = mfma(x, ones(NBF * SG + ch % SG / Q), accs[ch / SG]);
      }
    }
  };
  auto lds_barrier = []() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  // stage h is in LDS, the loads of stage h + AHEAD are under way; returns its
  // buffer. Rows past the samples hold dummy data: 0x80 bytes (0 after the XOR).
  auto arrive = [&](int h) {
    const int slot = h % NST;
    const int ahead = min(h + AHEAD - 1, nstage - 1) - h;
    if (more) wait_stage<C::LO + 1, NST>(ahead); else wait_stage<C::LO, NST>(ahead);
    asm volatile("s_barrier" ::: "memory");
    if (h + AHEAD < nstage) issue(h + AHEAD, (h + AHEAD) % NST);   // a buffer already read
    if (Lp - h * TR < TR) {
      const int rows = max(Lp - h * TR, 0), past = (TR - rows) * SEGS;
      uint8_t* buf = lds + slot * stage;
      for (int u = tid; u < nbeam * past; u += C::NTHR) {
        const int b = u / past, v = u % past;
        *(uint4*)(buf + 16 * ((b * UPB + rows * SEGS + v) ^ (b & 15))) =
            make_uint4(OFFSET_XOR, OFFSET_XOR, OFFSET_XOR, OFFSET_XOR);
      }
      lds_barrier();
    }
    return slot;
  };
  for (int h = 0; h < AHEAD && h < nstage; ++h) issue(h, h);
  for (int h = 0; h < nstage; h += 2) {
    constexpr std::integral_constant<int, 0> c0_{};
    constexpr std::integral_constant<int, 2> c2_{};
    constexpr std::integral_constant<int, 4> c4_{};
    uint32_t ol[NG][NBF][4], oh[NG][NBF][4], pl[NG][PG], ph[NG][PG];
    const int first = arrive(h);
    if constexpr (!C::PAIR) read_stage(first, c0_, c4_, ol, pl);
    const int slot = arrive(h + 1);
    if constexpr (C::PAIR) read_stage(first, c0_, c4_, ol, pl);
    if constexpr (C::HALVES) {
      read_stage(slot, c0_, c2_, oh, ph);
      multiply(c0_, c2_, ol, oh, pl, ph);
      asm volatile("" ::: "memory");
      read_stage(slot, c2_, c2_, oh, ph);
      multiply(c2_, c2_, ol, oh, pl, ph);
    } else {
      read_stage(slot, c0_, c4_, oh, ph);
      multiply(c0_, c4_, ol, oh, pl, ph);
    }
  }
  // every wave is past its last read of the ring before the epilogue reuses it
  lds_barrier();

  // the offset sums: the ones row's columns, or their own accumulators'
#pragma unroll
  for (int g = 0; g < NG * PG; ++g)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = 16 * NBF + (4 * kg + r) % RQ, ca = (4 * kg + r) / RQ;
      if constexpr (ONES) {
        if (16 * NBF + li % RQ == nbeam) {
#pragma unroll
          for (int b = 0; b < NBF; ++b)
            sxl[(16 * b + 4 * kg + r) * SXS + cb + g * Q + cs] = accp[g][b][r];
          if (ca == cs && a < nbeam) sxl[a * SXS + cb + g * Q + cs] = accr[g][r];
        }
      } else {
#pragma unroll
        for (int b = 0; b < NBF; ++b)
#pragma unroll
          for (int c = g * Q; c < g * Q + Q; ++c)
            if (li == b * SG + c % SG) sxl[(16 * b + 4 * kg + r) * SXS + cb + c] = accs[c / SG][r];
        if (li == NBF * SG + g * Q % SG / Q && a < nbeam)
          sxl[a * SXS + cb + g * Q + ca] = accs[g * Q / SG][r];
      }
    }
  const uint32_t cnt = (uint32_t)Lp;
  if (C::DIRECT && layout) {
    // cell records: the 16 lanes of a row hold consecutive pairs, which go
    // straight from the accumulators to the record, no staging in LDS
    lds_barrier();
    const bool shared = tl.parts > 1;
    auto put = [&](int32_t* dst, uint32_t raw) {
      if (shared) atomicAdd((unsigned*)dst, raw);   // integers: exact in any order
      else *dst = accumulate ? (int32_t)((uint32_t)*dst + raw) : (int32_t)raw;
    };
    const int nrow = nbeam + nbeam * (nbeam + 1) / 2;
    int32_t* tile = sum_x + ((int64_t)k * nchan + c0) * nrow;
    auto at = [&](int a) { return nbeam + a * nbeam - a * (a - 1) / 2 - a; };   // + b
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      if (c0 + cb + c >= nchan) continue;
      int32_t* rec = tile + (int64_t)(cb + c) * nrow;
      const int32_t* sx = sxl + cb + c;
      uint32_t sb[NBF];
#pragma unroll
      for (int b = 0; b < NBF; ++b) sb[b] = 128u * (uint32_t)sx[(16 * b + li) * SXS];
#pragma unroll
      for (int b1 = 0; b1 < NBF; ++b1)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * b1 + 4 * kg + r;
          const uint32_t sa = 128u * (uint32_t)sx[a * SXS] + 16384u * cnt;
#pragma unroll
          for (int b2 = b1; b2 < NBF; ++b2)
            if (b2 > b1 || 4 * kg + r <= li)
              put(rec + at(a) + 16 * b2 + li,
                  (uint32_t)acc[c][block_pair(b1, b2, NBF)][r] + sa + sb[b2]);
        }
    }
    const int b = 16 * NBF + li % RQ;
#pragma unroll
    for (int g = 0; g < NG * PG; ++g) {
      const int ch = cb + g * Q + cs;
      if (b >= nbeam || c0 + ch >= nchan) continue;
      int32_t* rec = tile + (int64_t)ch * nrow;
      const int32_t* sx = sxl + ch;
      const uint32_t sb = 128u * (uint32_t)sx[b * SXS] + 16384u * cnt;
#pragma unroll
      for (int b1 = 0; b1 < NBF; ++b1)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * b1 + 4 * kg + r;
          put(rec + at(a) + b, (uint32_t)accp[g][b1][r] + 128u * (uint32_t)sx[a * SXS] + sb);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * NBF + (4 * kg + r) % RQ;
        if ((4 * kg + r) / RQ == cs && a <= b)
          put(rec + at(a) + b, (uint32_t)accr[g][r] + 128u * (uint32_t)sx[a * SXS] + sb);
      }
    }
    for (int i = tid; i < nbeam * CW; i += C::NTHR) {
      const int ch = i / nbeam, a = i % nbeam;
      if (c0 + ch < nchan)
        put(tile + (int64_t)ch * nrow + a, (uint32_t)sxl[a * SXS + ch] + 128u * cnt);
    }
    nh = 0;                                    // stored
  }
  const int cwp = CW / max(nh, 1);
  for (int h = 0; h < nh; ++h) {
    if (cb / cwp == h) {
      int32_t* st = stg + (cb - h * cwp);
      auto row_of = [&](int a, int b) { return a * nbeam - a * (a - 1) / 2 + (b - a); };
#pragma unroll
      for (int b1 = 0; b1 < NBF; ++b1)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * b1 + 4 * kg + r;
#pragma unroll
          for (int b2 = b1; b2 < NBF; ++b2) {
            const int b = 16 * b2 + li;
            if (a <= b) {
              int32_t* dst = st + row_of(a, b) * (cwp + 1);
#pragma unroll
              for (int c = 0; c < CPW; ++c) dst[c] = acc[c][block_pair(b1, b2, NBF)][r];
            }
          }
          const int b = 16 * NBF + li % RQ;
          if (b < nbeam) {
            int32_t* dst = st + row_of(a, b) * (cwp + 1) + cs;
#pragma unroll
            for (int g = 0; g < NG * PG; ++g) dst[g * Q] = accp[g][b1][r];
          }
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * NBF + (4 * kg + r) % RQ, b = 16 * NBF + li % RQ;
        if ((4 * kg + r) / RQ == cs && a <= b && b < nbeam) {
          int32_t* dst = st + row_of(a, b) * (cwp + 1) + cs;
#pragma unroll
          for (int g = 0; g < NG * PG; ++g) dst[g * Q] = accr[g][r];
        }
      }
    }
    lds_barrier();
    store_sums(stg, sxl, nbeam, SXS, cwp, h, c0, nchan, k, ncell, layout, sum_x, sum_xy,
               cnt, tl.parts > 1, accumulate, tid, C::NTHR);
    lds_barrier();
  }
  if (c0 == 0 && tl.part == 0 && tid == 0) {
    const int Lk = k % ksplit == ksplit - 1 ? Llast : L;
    count[k] = accumulate ? count[k] + Lk : Lk;
  }
}

// Epilogue passes: the fewest (power of two, whole waves each) whose staging
// rows fit; 0 if none does.
template <int NB, int CW, int CPW, int IPW, int NST>
int epilogue_passes(int nbeam) {
  using C = MfmaCfg<NB, CW, CPW, IPW, NST>;
  const int np = nbeam * (nbeam + 1) / 2;
  int nh = 1;
  while (nh < C::NWAVE && np * (CW / nh + 1) * 4 > C::STG_BYTES) nh *= 2;
  return np * (CW / nh + 1) * 4 > C::STG_BYTES ? 0 : nh;
}

// Zeroes cells [first, ncell) of the outputs (those of a launch in parts).
__global__ __launch_bounds__(256) void zero_kernel(int32_t* a, int64_t rows_a, int32_t* b,
                                                   int64_t rows, int64_t ld, int64_t first) {
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
    int32_t* p = r < rows_a ? a + r * ld : b + (r - rows_a) * ld;
    for (int64_t i = first + (int64_t)blockIdx.x * 256 + threadIdx.x; i < ld; i += step) p[i] = 0;
  }
}
hipError_t launch_zero(int32_t* sum_x, int32_t* sum_xy, int nbeam, int64_t ncell, int64_t first,
                       int layout, hipStream_t s) {
  const int64_t np = npair_of(nbeam), nrow = nbeam + np;
  const int64_t rows = layout ? 1 : nrow, ld = layout ? ncell * nrow : ncell;
  const int64_t off = layout ? first * nrow : first;
  int64_t bx = (ld - off + 2047) / 2048;
  if (bx > 2048) bx = 2048;
  int64_t by = rows < 2048 / bx ? rows : 2048 / bx;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)bx, (unsigned)(by < 1 ? 1 : by)), dim3(256), 0, s,
                     sum_x, layout ? rows : nbeam, sum_xy, rows, ld, off);
  return hipGetLastError();
}
// the outputs of the batched items in parts
__global__ __launch_bounds__(256) void zero_items_kernel(const CcmItem* items) {
  const CcmItem& it = items[blockIdx.y];
  if (it.parts == 1) return;
  const int64_t ncell = (int64_t)it.nsub * it.nchan, np = (int64_t)it.nbeam * (it.nbeam + 1) / 2;
  const int64_t na = ncell * (it.layout ? it.nbeam + np : it.nbeam), nb = it.layout ? 0 : ncell * np;
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < na + nb; i += step)
    *(i < na ? it.sum_x + i : it.sum_xy + (i - na)) = 0;
}

// How a launch of ntiles tiles of L samples meets `slots` workgroup slots: one
// that leaves CUs idle, or whose last round does, shares the samples of the last
// round's tiles out. Cost in chunks per slot: rounds x (chunks + epilogue), for
// the shared ones with a zeroing launch and atomic stores in place of plain
// ones; shared only for a gain of a fiftieth. epilogue: chunks that a shared one
// costs, 12, or where records go straight to memory what the atomics of all
// nbeam + npair rows cost at one per ns and CU (72 beams 34: 4096 channels x 700
// samples, 128 tiles, in 2 parts 196 us, whole 143 us). 19 beams: 16 tiles of
// 1024 samples in 8 parts 49 -> 20 us (and 3 us to zero).
template <class C>
int shared_epilogue(int nbeam) {
  return C::DIRECT ? 6 + (nbeam + 3) * 3 / 8 : 12;
}

}  // namespace

CcmShare ccm_share(int64_t ntiles, int L, int slots, int epilogue) {
  const int nchunk = (L + TC - 1) / TC;
  const int64_t full = ntiles / slots, tail = ntiles - full * slots;
  CcmShare sh{(int)ntiles, 1, (full + (tail > 0)) * (nchunk + 8)};
  if (tail == 0 || nchunk < 8) return sh;
  int64_t best = sh.cost * 49 / 50;
  for (int p = 2; p <= 32 && p * 4 <= nchunk; ++p) {
    const int64_t cost = full * (nchunk + 8) +
                         (tail * p + slots - 1) / slots * ((nchunk + p - 1) / p + epilogue) + 4;
    if (cost < best) {
      best = cost;
      sh = CcmShare{(int)(full * slots), p, cost};
    }
  }
  return sh;
}

namespace {

template <class C, class K>
hipError_t launch_cfg(K kern, int nh, const BeamPtrs& bp, int nbeam, int nchan, int64_t row_stride,
                           int64_t t0, int L, int nsub, int32_t* sum_x, int32_t* sum_xy,
                           int32_t* count, int accumulate, int group_bytes, int layout,
                           int64_t kstride, int ksplit, int Llast, hipStream_t s) {
  if ((int64_t)nbeam * C::UPB * 16 > C::STAGE || nbeam > C::MAXB || nh == 0) return hipErrorInvalidValue;
  const int nct = (nchan + C::WIDTH - 1) / C::WIDTH;
  hipError_t e = hipFuncSetAttribute((const void*)kern,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
  if (e != hipSuccess) return e;
  const int64_t ntiles = (int64_t)nsub * nct;
  const CcmShare sh = ksplit > 1 ? CcmShare{(int)ntiles, 1, 0}
                                 : ccm_share(ntiles, L, C::SLOTS, shared_epilogue<C>(nbeam));
  const int64_t nshared = (ntiles - sh.nwhole) * sh.parts;
  const int G = group_tiles(C::WIDTH, group_bytes, sh.nwhole) |
                group_tiles(C::WIDTH, group_bytes, nshared) << 16;
  if (sh.parts > 1 && !accumulate) {
    e = launch_zero(sum_x, sum_xy, nbeam, (int64_t)nsub * nchan,
                    (int64_t)(sh.nwhole / nct) * nchan, layout, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(sh.nwhole + nshared)),
                     dim3(C::NTHR), C::LDS, s, bp, nbeam, nchan, row_stride, t0, L, nsub, nct, sum_x,
                     sum_xy, count, accumulate, G, nh, layout, kstride, ksplit, Llast,
                     sh.nwhole, sh.parts, (const CcmItem*)nullptr, 0);
  return hipGetLastError();
}

template <class C, class K>
hipError_t launch_batch_cfg(K kern, const CcmItem* items, int nitem, int total_wg, int group_bytes,
                            hipStream_t s) {
  hipError_t e = hipFuncSetAttribute((const void*)kern,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
  if (e != hipSuccess) return e;
  const int G = group_tiles(C::WIDTH, group_bytes, INT64_MAX);
  BeamPtrs none;
  memset(&none, 0, sizeof(none));
  hipLaunchKernelGGL(kern, dim3((unsigned)total_wg), dim3(C::NTHR), C::LDS, s, none, 0, 0,
                     (int64_t)0, (int64_t)0, 0, 0, 0, (int32_t*)nullptr, (int32_t*)nullptr,
                     (int32_t*)nullptr, 0, G, 1, 0, (int64_t)0, 1, 0, 0, 1, items, nitem);
  return hipGetLastError();
}

// Largest ring (<= 4 buffers) of IPW KB-per-wave chunk buffers within 160 KB;
// calls op.run<config>(kernel, epilogue passes).
template <int NB, int CW, int CPW, int IPW, class Op>
hipError_t dispatch_nst(int nbeam, int max_stages, Op& op) {
#define RFI_NST(NST)                                                              \
  if constexpr (MfmaCfg<NB, CW, CPW, IPW, NST>::FITS) {                             \
    if (max_stages >= NST)                                                        \
      return op.template run<MfmaCfg<NB, CW, CPW, IPW, NST>>(                       \
          ccm_mfma_kernel<NB, CW, CPW, IPW, NST>, epilogue_passes<NB, CW, CPW, IPW, NST>(nbeam)); \
  }
  RFI_NST(4) RFI_NST(3) RFI_NST(2)
#undef RFI_NST
  return hipErrorInvalidValue;
}

// The packed engine's instance for a beam count it takes: Q = 4 channels per
// packed operand where the beams left and the ones row fit in 4 rows, else 2.
template <class Op>
hipError_t pack_dispatch(int nbeam, Op& op) {
  const int nbf = nbeam / 16, left = nbeam % 16;
#define RFI_PACK(NBF, Q, ONES)                                                          \
  if (nbf == NBF && (left <= 3 ? 4 : 2) == Q && (left < 8) == ONES)                     \
    return op.template run<PackCfg<NBF, Q, ONES>>(ccm_pack_kernel<NBF, Q, ONES>,          \
                                                  PackCfg<NBF, Q, ONES>::passes(nbeam));
  RFI_PACK(1, 4, true)
  RFI_PACK(2, 4, true) RFI_PACK(2, 2, true) RFI_PACK(2, 2, false)
  RFI_PACK(3, 4, true) RFI_PACK(3, 2, true) RFI_PACK(3, 2, false)
  RFI_PACK(4, 4, true) RFI_PACK(4, 2, true) RFI_PACK(4, 2, false)
#undef RFI_PACK
  return hipErrorInvalidValue;
}

// Whether a launch over `cells` (sub-interval, channel) cells of L samples takes
// the packed engine. Its tiles are as wide or wider on fewer waves, so they have to
// fill the chip (whole blocks -> packed, us):
//   32..72 beams (16 k to 16 k + 8): tiles of twice the channels, 128 of them (from 48
//     beams on 96), and up to 1024 samples, where a round (256 tiles) is mostly
//     epilogue, fewer rounds than whole blocks need: 48 beams x 1000 channels, 161
//     samples x 8 (256 tiles, whole blocks 504) 97 -> 36; 35 x 2048, 697 x 4 (128,
//     256) 51 -> 64; 48 x 4096, 482 x 1 (128, 256) 48 -> 54.
//   68..72 beams, whose packed step and epilogue cost more (operands in scratch, two
//     accumulators more per channel pair): rounds x (chunks + 11) 5 / 4 against
//     rounds x (chunks + 5), up to 4096 samples. 72 beams: 1000 x 300 x 9 (288
//     tiles, 567) 202 -> 272, 2000 x 87 x 21 549 -> 662, 2048 x 340 x 19 961 -> 832,
//     1024 x 2048 x 4 309 -> 443, x 8000 x 4 1074 -> 922.
//   16..19 beams, where only the epilogues are overlapped (two workgroups per CU):
//     768 tiles of up to 1024 samples; of up to 3072 by the rounds that either needs
//     (CcmShare::cost): a packed one, of twice the workgroups, takes 2 x (0.875 +
//     samples / 65536) whole ones. packed / whole, 19 beams x 4096 channels: 832
//     tiles (3.25 whole rounds, the last one shared out) of 1100 / 1500 / 2000 / 3000
//     samples 0.96 / 0.99 / 1.02 / 1.02, 960 tiles 0.92 / 0.94 / 0.94 / 0.97, 3200
//     tiles 0.92 / 0.93 / 0.95 / 0.98; 1536 of 8192 1.02, 640 of 20345 1.12 (the
//     neighbouring workgroups that share 128-byte lines drift apart). Lined-up beams
//     (ccm_lined_up) queue on the same memory channels however the epilogues lie: up
//     to 512 samples there (832 tiles: 512 147 -> 138 us, 1024 246 -> 256, 2048 456
//     -> 494).
bool takes_pack(int nbeam, const CcmTune* t, int64_t cells, int L, bool lined) {
  if (t && (t->tile || t->stages || t->engine == 1)) return false;   // a choice of the other
  const int nbf = nbeam / 16, left = nbeam % 16;
  if (nbf < 1 || nbf > 4 || left > (nbf == 1 ? 3 : 8)) return false;
  if (t && t->engine == 2) return true;
  if (nbf == 1) {
    if (cells < 768 * 64 || L > (lined ? 512 : 3072)) return false;
    if (L <= 1024) return true;
    const int64_t tiles = std::min<int64_t>(cells, (int64_t)1 << 40) / 64;
    return ccm_share(tiles, L, 512, 12).cost * 2 * (57344 + L) <
           ccm_share(tiles, L, 256, 12).cost * 65536;
  }
  if (cells < (nbf == 2 ? 128 * 64 : 96 * 32)) return false;
  const int64_t per = 256 * (nbf == 2 ? 64 : 32);       // cells of a packed round
  const int64_t most = std::min<int64_t>(cells, (int64_t)1 << 40);
  const int64_t packed = (most + per - 1) / per, whole = (2 * most + per - 1) / per;
  const int nchunk = (L + TC - 1) / TC;
  if (nbf == 4 && left >= 4)
    return L > 4096 || packed * 5 * (nchunk + 11) < whole * 4 * (nchunk + 5);
  return L > 1024 || packed < whole;
}

// The MFMA engine's instance for a beam count: 16-row blocks NB (including
// the ones row), tile width CW channels, CPW channels per wave, IPW loads per
// wave per chunk, ring depth NST. t (nullable) selects another tile variant
// of the beam count and caps the ring depth.
template <class Op>
hipError_t ccm_dispatch(int nbeam, int shared_cu, bool pack, Op& op, const CcmTune* t) {
  const int nb = (nbeam + 1 + 15) / 16;
  // tile shape per block count: (CW channels, CPW channels per wave). The
  // 16-31-beam default is 64 channels on 16 waves of 4 channels (a 3-deep
  // ring of 48 KB chunks): on the 19-beam FAST block it beats 8 waves of 8
  // channels (4-deep ring), variant 1, by about 3 % once the beams are
  // staggered across the memory channels. With shared_cu the tile is 32
  // channels on 8 waves of ~120 VGPRs.
  int cw, cpw;
  const int tile = t ? t->tile : 0;
  if (tile < 0 || tile >= ccm_tile_variants(nbeam)) return hipErrorInvalidValue;
  if (pack) return pack_dispatch(nbeam, op);
  switch (nb) {
    case 1: cw = 64; cpw = 8; break;
    case 2:
      if (tile == 1) { cw = 64; cpw = 8; }
      else if (tile == 2 || shared_cu) { cw = 32; cpw = 4; }
      else { cw = 64; cpw = 4; }
      break;
    case 3: cw = 32; cpw = 4; break;
    case 4: case 5: cw = 16; cpw = 2; break;
    default: return hipErrorInvalidValue;
  }
  // ring depth cap (a tune entry's choice; default: the largest ring that fits)
  const int max_stages = t && t->stages >= 2 ? t->stages : 4;
  const int nwave = cw / cpw;
  const int units = nbeam * 32 * (cw / 16);        // 16-byte units per chunk
  const int ipw = (units + 64 * nwave - 1) / (64 * nwave);  // loads per wave per chunk
#define RFI_CCM(NB, CW, CPW, IPW)                         \
  if (nb == NB && cw == CW && cpw == CPW && ipw == IPW) \
    return dispatch_nst<NB, CW, CPW, IPW>(nbeam, max_stages, op);
  RFI_CCM(1, 64, 8, 1) RFI_CCM(1, 64, 8, 2) RFI_CCM(1, 64, 8, 3) RFI_CCM(1, 64, 8, 4)
  RFI_CCM(2, 64, 8, 4) RFI_CCM(2, 64, 8, 5) RFI_CCM(2, 64, 8, 6) RFI_CCM(2, 64, 8, 7)
  RFI_CCM(2, 64, 8, 8)
  RFI_CCM(2, 64, 4, 2) RFI_CCM(2, 64, 4, 3) RFI_CCM(2, 64, 4, 4)
  RFI_CCM(2, 32, 4, 2) RFI_CCM(2, 32, 4, 3) RFI_CCM(2, 32, 4, 4)
  RFI_CCM(3, 32, 4, 4) RFI_CCM(3, 32, 4, 5) RFI_CCM(3, 32, 4, 6)
  RFI_CCM(4, 16, 2, 3) RFI_CCM(4, 16, 2, 4)
  RFI_CCM(5, 16, 2, 4) RFI_CCM(5, 16, 2, 5)
#undef RFI_CCM
  return hipErrorInvalidValue;
}

struct LaunchOne {
  const BeamPtrs& bp;
  int nbeam, nchan;
  int64_t row_stride, t0;
  int L, nsub;
  int32_t *sum_x, *sum_xy, *count;
  int accumulate, group_bytes, layout;
  int64_t kstride;
  int ksplit, Llast;
  hipStream_t s;
  template <class C, class K>
  hipError_t run(K kern, int nh) {
    return launch_cfg<C>(kern, nh, bp, nbeam, nchan, row_stride, t0, L, nsub, sum_x, sum_xy, count,
                         accumulate, group_bytes, layout, kstride, ksplit, Llast, s);
  }
};

struct Describe {
  int nbeam;
  CcmClass* out;
  template <class C, class K>
  hipError_t run(K, int nh) {
    out->key = C::KEY;
    out->cw = C::WIDTH;
    out->nh = nh;
    out->slots = C::SLOTS;
    out->epilogue = shared_epilogue<C>(nbeam);
    return nh > 0 ? hipSuccess : hipErrorInvalidValue;
  }
};

struct LaunchBatch {
  const CcmItem* items;
  int nitem, total_wg, group_bytes;
  hipStream_t s;
  template <class C, class K>
  hipError_t run(K kern, int) {
    return launch_batch_cfg<C>(kern, items, nitem, total_wg, group_bytes, s);
  }
};

// ---------------------------------------------------------------------------
// VALU comparison engine: one lane per channel, nbeam <= 20.
constexpr int VN = 20;
constexpr int VNP = VN * (VN + 1) / 2;

__global__ __launch_bounds__(256) void ccm_valu_kernel(BeamPtrs bp, int nbeam, int nchan,
                                                       int64_t row_stride, int64_t t0, int L,
                                                       int nsub, int32_t* __restrict__ sum_x,
                                                       int32_t* __restrict__ sum_xy,
                                                       int32_t* __restrict__ count,
                                                       int accumulate) {
  const int chan = blockIdx.x * 256 + threadIdx.x;
  const int k = blockIdx.y;
  if (blockIdx.x == 0 && threadIdx.x == 0) count[k] = accumulate ? count[k] + L : L;
  if (chan >= nchan) return;
  const int64_t row0 = t0 + (int64_t)k * L;
  uint32_t acc[VNP];
  uint32_t sx[VN];
#pragma unroll
  for (int i = 0; i < VNP; ++i) acc[i] = 0;
#pragma unroll
  for (int i = 0; i < VN; ++i) sx[i] = 0;
  for (int t = 0; t < L; t += 4) {
    uint32_t x[VN];
#pragma unroll
    for (int b = 0; b < VN; ++b) {
      uint32_t v = 0;
      if (b < nbeam) {
        const uint8_t* p = bp.p[b] + (row0 + t) * row_stride + chan;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t + i < L) v |= (uint32_t)p[i * row_stride] << (8 * i);
      }
      x[b] = v;
    }
#pragma unroll
    for (int a = 0; a < VN; ++a) {
      sx[a] = __builtin_amdgcn_udot4(x[a], 0x01010101u, sx[a], false);
#pragma unroll
      for (int b = a; b < VN; ++b) {
        const int idx = a * VN - a * (a - 1) / 2 + (b - a);
        acc[idx] = __builtin_amdgcn_udot4(x[a], x[b], acc[idx], false);
      }
    }
  }
  const int64_t ncell = (int64_t)nsub * nchan;
  const int64_t cell = (int64_t)k * nchan + chan;
#pragma unroll
  for (int a = 0; a < VN; ++a) {
    if (a >= nbeam) continue;
    int32_t* d = sum_x + a * ncell + cell;
    *d = accumulate ? (int32_t)((uint32_t)*d + sx[a]) : (int32_t)sx[a];
#pragma unroll
    for (int b = a; b < VN; ++b) {
      if (b >= nbeam) continue;
      const int idx = a * VN - a * (a - 1) / 2 + (b - a);
      const int64_t out = (int64_t)a * nbeam - (int64_t)a * (a - 1) / 2 + (b - a);
      int32_t* q = sum_xy + out * ncell + cell;
      *q = accumulate ? (int32_t)((uint32_t)*q + acc[idx]) : (int32_t)acc[idx];
    }
  }
}

}  // namespace

int ccm_tile_variants(int nbeam) {
  const int nb = (nbeam + 1 + 15) / 16;
  return nb == 2 ? 3 : (nb >= 1 && nb <= 5 ? 1 : 0);
}

bool ccm_lined_up(const uint8_t* const* beam, int nbeam, int64_t row_stride) {
  if (row_stride % 1024) return false;
  for (int b = 1; b < nbeam; ++b)
    if (((uintptr_t)beam[b] ^ (uintptr_t)beam[0]) & 4095) return false;
  return true;
}

hipError_t launch_ccm_mfma(const BeamPtrs& bp, int nbeam, int nchan, int64_t row_stride,
                           int64_t t0, int L, int nsub, int32_t* sum_x, int32_t* sum_xy,
                           int32_t* count, int accumulate, int shared_cu, hipStream_t s,
                           const CcmTune* t, int layout, int64_t kstride, int ksplit, int Llast) {
  LaunchOne op{bp, nbeam, nchan, row_stride, t0, L, nsub, sum_x, sum_xy, count, accumulate,
               t ? t->group_bytes : 0, layout, kstride, ksplit, Llast, s};
  const bool pack = !shared_cu && takes_pack(nbeam, t, (int64_t)nsub * nchan, L,
                                             ccm_lined_up(bp.p, nbeam, row_stride));
  return ccm_dispatch(nbeam, shared_cu, pack, op, t);
}

hipError_t launch_ccm_mfma(const BeamPtrs& bp, int nbeam, int nchan, int64_t row_stride,
                           int64_t t0, int L, int nsub, int32_t* sum_x, int32_t* sum_xy,
                           int32_t* count, int accumulate, int shared_cu, hipStream_t s,
                           const CcmTune* t, int layout, int64_t kstride, int ksplit) {
  return launch_ccm_mfma(bp, nbeam, nchan, row_stride, t0, L, nsub, sum_x, sum_xy, count,
                         accumulate, shared_cu, s, t, layout, kstride, ksplit, L);
}

hipError_t ccm_class(int nbeam, CcmClass* c, const CcmTune* t, int64_t cells, int L, bool lined) {
  Describe op{nbeam, c};
  const bool pack = takes_pack(nbeam, t, cells, L, lined);
  c->engine = pack ? 2 : 1;
  hipError_t e = ccm_dispatch(nbeam, 0, pack, op, t);
  // the tile group size is a launch argument: part of the class
  c->group_bytes = t ? t->group_bytes : 0;
  c->key = c->key * 65536 + (c->group_bytes & 0xFFFF);   // (instance, group)
  return e;
}

int ccm_chunks(int L) { return (L + TC - 1) / TC; }

hipError_t launch_ccm_batch(int nbeam_of_class, const CcmTune* t, const CcmItem* items,
                            int nitem, int total_wg, bool parts, hipStream_t s) {
  if (parts)
    hipLaunchKernelGGL(zero_items_kernel, dim3(256, (unsigned)nitem), dim3(256), 0, s, items);
  LaunchBatch op{items, nitem, total_wg, t ? t->group_bytes : 0, s};
  return ccm_dispatch(nbeam_of_class, 0, t && t->engine == 2, op, t);
}

hipError_t launch_ccm_valu(const BeamPtrs& bp, int nbeam, int nchan, int64_t row_stride,
                           int64_t t0, int L, int nsub, int32_t* sum_x, int32_t* sum_xy,
                           int32_t* count, int accumulate, hipStream_t s) {
  if (nbeam > VN) return hipErrorInvalidValue;
  dim3 grid((nchan + 255) / 256, nsub);
  hipLaunchKernelGGL(ccm_valu_kernel, grid, dim3(256), 0, s, bp, nbeam, nchan, row_stride, t0,
                     L, nsub, sum_x, sum_xy, count, accumulate);
  return hipGetLastError();
}

}  // namespace rfi
