// How the 64-row attention kernels lay out a tile in LDS and share out their
// work: plain C++ (no device code), so the index tests compile and call these
// very functions.
#pragma once

namespace smem {

constexpr int BT = 64;         // block / page size of the MFMA attention kernels

// Tile of workgroup n of `all` when each XCD (workgroup index mod 8) takes a
// contiguous range of them: a permutation of 0 .. all - 1.
constexpr int xcd_range(int n, int all) {
  const int x = n & 7, more = all & 7;
  return x * (all >> 3) + (x < more ? x : more) + (n >> 3);
}

// The key of a 64-key tile that a lane's score s[kt][i] belongs to, less the
// lane's own part 8 (lane / 16): the two 16-row score tiles of 32 keys
// interleave by fours (tile_row below), so the lane's scores of tiles 2c and
// 2c + 1 are 8 consecutive keys.
constexpr int score_key(int kt, int i) { return (kt >> 1) * 32 + (kt & 1) * 4 + i; }

// ------------------------------------------------------------------ LDS tile layout

// A 64-key tile in LDS -- a memory page's (page, head) tile, or a block's own
// keys and values -- keeps the page layout: the key plane [b][d_h] followed by
// the transposed value plane [d_h][b], with the 16-byte slots of each row
// permuted (key row r: slot = chunk ^ kswz(r); value row d: slot = chunk ^
// vswz(d)), so the rows one MFMA operand read touches fall on distinct banks
// (measured on gfx950: no bank conflicts for the key and value operand reads).
// The key rows of each 32 are reordered by fours (key 8g + 4h + i in row 16h +
// 4g + i): a lane's weights of two score tiles then belong to 8 consecutive
// keys, and its value operand is one 16-byte read where it was two of 8.
// Memory pages of the non-rotary prefill move global -> LDS by DMA
// (global_load_lds_dwordx4, 16 bytes per lane) through a ring of NS page
// stages, so NS - 1 pages are in flight while one is read and no register
// holds a page in transit.
#ifndef SMEM_PREFILL_STAGES32
#define SMEM_PREFILL_STAGES32 4
#endif
#ifndef SMEM_PREFILL_STAGES64
#define SMEM_PREFILL_STAGES64 4
#endif
#ifndef SMEM_PREFILL_STAGES128
#define SMEM_PREFILL_STAGES128 2
#endif
template <int DH>
struct PageRing {
  static constexpr int TILE = 2 * BT * DH * 2;         // bytes per (page, head)
  static constexpr int KBYTES = BT * DH * 2;           // key plane bytes
  static constexpr int KRB = DH * 2;                   // key row bytes
  static constexpr int KCH = DH / 8;                   // 16-byte chunks per key row
  static constexpr int NS = DH == 32 ? SMEM_PREFILL_STAGES32 : DH == 64 ? SMEM_PREFILL_STAGES64 : SMEM_PREFILL_STAGES128;
  static constexpr int IPW = TILE / 1024 / 4;          // DMA instructions per wave per page
  static_assert(NS >= 2 && NS <= 5, "wait_pages covers up to 3 pages ahead");
  // key rows: slot = chunk ^ kswz(r).  Chosen by measurement (a one-wave LDS
  // bank probe of the score reads): r / 2 for 64-byte rows (r / 4 left them
  // 2-way conflicted), r / 2 for 128-byte rows, r for 256-byte rows.
  static constexpr int kswz(int r) { return (DH == 32 ? r / 2 : r / (256 / KRB)) % KCH; }
  // value rows: 16 rows of 128 bytes per operand read, as the keys at d_h = 64.
  // At d_h = 128 the row group is added: a block's own values are written 16
  // chunks of a row pair at a time, which d / 2 alone puts on two slots (8
  // ways; encoder, 30 blocks of 20 heads 8.6 us against 8.9).  Below that one
  // operand address for all row groups is worth more (d_h 64, 128 blocks of
  // 12 heads: 9.2 us against 9.6).
  static constexpr int vswz(int d) { return ((d >> 1) ^ (DH == 128 ? d >> 4 : 0)) & 7; }
  // LDS row of a key of the tile, and the key in an LDS row
  static constexpr int tile_row(int key) {
    return (key & ~31) + ((key >> 2) & 1) * 16 + ((key >> 3) & 3) * 4 + (key & 3);
  }
  static constexpr int row_key(int row) {
    return (row & ~31) + ((row >> 2) & 3) * 8 + ((row >> 4) & 1) * 4 + (row & 3);
  }
  // LDS byte of chunk c (8 dims) of the key in LDS row r, and of the 32-bit
  // pair of value dim d that starts at the even key `key`
  static constexpr int key_at(int r, int c) { return r * KRB + ((c ^ kswz(r)) << 4); }
  static constexpr int value_at(int d, int key) {
    return KBYTES + d * 128 + (key & 7) * 2 + (((key >> 3) ^ vswz(d)) << 4);
  }
  // LDS bytes of the 8 keys 8 (l / 16) + 32 c .. +7 of value row dt * 16 + l %
  // 16, a lane's value operand: one address per lane, the rest constants
  static constexpr int operand_lane(int lane) {
    return KBYTES + (lane & 15) * 128 + (((lane >> 4) ^ vswz(lane & 15)) << 4);
  }
  static constexpr int operand_at(int lane_byte, int dt, int c) {
    return (lane_byte ^ (vswz(dt * 16) << 4) ^ (c * 64)) + dt * 2048;
  }
  // Byte of the (page, head) tile in memory that LDS byte `byte` holds.
  static constexpr int source(int byte) {
    if (byte < KBYTES) {
      const int r = byte / KRB, sl = (byte % KRB) >> 4;
      return row_key(r) * KRB + ((sl ^ kswz(r)) << 4);
    }
    const int vb = byte - KBYTES, d = vb >> 7, sl = (vb & 127) >> 4;
    return KBYTES + d * 128 + ((sl ^ vswz(d)) << 4);
  }
};

// ------------------------------------------------------------------ few-pair prefill

constexpr int kParSplits = 4;  // memory splits that the few-pair variant reads at once

template <int DH, int QW>
struct ParLds {
  using R = PageRing<DH>;
  static constexpr int G = kParSplits;                 // split groups
  static constexpr int NSP = DH == 32 ? 4 : 2;         // ring stages per group
  static constexpr int IPW = R::TILE / 1024 / QW;      // DMA instructions per wave per page
  static constexpr int THREADS = 64 * G * QW;
  static constexpr int ROWS = 16 * QW;                 // query rows per workgroup
  static constexpr int RING = G * NSP * R::TILE;
  static constexpr int OFF_IN = RING;                  // in-block tile, ring layout
  static constexpr int OFF_NULL = OFF_IN + R::TILE;    // null key, then null value (bf16)
  static constexpr int BYTES = OFF_NULL + 4 * DH;
  // a split state per (slot, wave): o as DH/16 float4 planes of 64 lanes, then (m, l) pairs;
  // slots 0..3 hold memory splits 0..3, slot 4 the final split
  static constexpr int STATE = (DH / 16) * 1024 + 64 * 8;
  static_assert((G + 1) * QW * STATE <= RING, "split states fit in the ring");
  static_assert(BYTES <= 160 * 1024, "LDS");
  static_assert(NSP >= 2 && NSP <= 4 && 3 * IPW < 64, "wait_pages covers up to 3 pages ahead");
};

// Query-row waves per split group: up to 64 pairs, four workgroups of 16 rows
// still run one per CU: us per call over 15 pages on 1 / 2: 32 heads of 32, 1
// block 6.8 / 7.9, 4 blocks 12.8 / 9.0; 16 heads of 64, 1 block 8.4 / 9.8; 12
// heads, 8 blocks 19.1 / 12.6.
constexpr int par_row_waves(int n_pairs) { return n_pairs <= 64 ? 1 : 2; }
// Workgroups of a few-pair launch: 4/QW parts per pair, 8 pairs per round of
// 8 x (4/QW) launch indices, so the parts of a pair run on one XCD.
constexpr int par_grid(int n_pairs, int qw) { return ((n_pairs + 7) / 8) * 8 * (4 / qw); }
constexpr int par_pair(int n, int qw) { return (n / (8 * (4 / qw))) * 8 + n % 8; }
constexpr int par_part(int n, int qw) { return (n / 8) % (4 / qw); }

}  // namespace smem
