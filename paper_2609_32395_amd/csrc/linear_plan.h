// How a linear map is cut into workgroups: which kernel and tile a size gets,
// how much LDS a launch takes, which tile a workgroup computes, and where a
// tile's values lie in LDS.  Plain C++ (no device code), so the index tests
// compile and call these very functions.
#pragma once

namespace smem {

constexpr long ceil_div(long a, long b) { return (a + b - 1) / b; }

// The chunk that a reduction over K is cut into (linear.h, the reduction order).
constexpr int lin_chunk(int K) { return 256 * ((K + 256 * 16 - 1) / (256 * 16)); }
constexpr int lin_chunks(int K) { return (K + lin_chunk(K) - 1) / lin_chunk(K); }

// Launch order -> work item.  Workgroups are dealt to the 8 XCDs round-robin
// (workgroup i to XCD i mod 8); the grid is padded to a multiple of 8 and
// item p = (i mod 8) * (T8 / 8) + i / 8, so each XCD takes one contiguous
// range of items and neighbouring items share that XCD's L2.  Padding
// workgroups get -1 and exit.
constexpr int xcd_grid(int T) { return (T + 7) & ~7; }
constexpr int xcd_order(int i, int T) {
  const int p = (i & 7) * (xcd_grid(T) >> 3) + (i >> 3);
  return p < T ? p : -1;
}

// ---------------------------------------------------------------- few rows

// A wave's 16-row, 256-wide piece in LDS: row r is 32 slots of 16 bytes, chunk
// q in slot q ^ r, so the 16 rows one operand read touches lie on distinct
// banks.
struct FewTile {
  static constexpr int BYTES = 8192;
  // write: instruction i of a half-wave holds row r, chunk s = lane % 32
  static constexpr int put(int r, int s) { return r * 512 + ((s ^ r) << 4); }
  // operand of step t: lane (row l % 16, group l / 16) reads chunk 4 t + group
  static constexpr int get(int lane, int t) {
    return (lane & 15) * 512 + (((t * 4 + (lane >> 4)) ^ (lane & 15)) << 4);
  }
};

// The maps without a LayerNorm: row tiles x column tiles of 16, waves, and
// whether a wave takes several pieces of K.
struct FewPlan {
  int rt, g, nw;
  bool loop;
};
constexpr FewPlan kFewPlans[] = {{1, 1, 8, false}, {2, 2, 8, false}, {2, 4, 8, false}, {1, 1, 16, false},
                                 {2, 1, 16, false}, {1, 1, 8, true}, {1, 2, 8, true}};
enum FewKind { kFew1x1, kFew2x2, kFew2x4, kFewDeep1x1, kFewDeep2x1, kFewLong1x1, kFewLong1x2 };
constexpr int few_waves(const FewPlan& p, int K) { return lin_chunks(K) < p.nw ? lin_chunks(K) : p.nw; }
constexpr long few_lds_bytes(const FewPlan& p, int K) {
  return (long)few_waves(p, K) * FewTile::BYTES + (long)lin_chunks(K) * p.rt * p.g * 1024;
}

// The tile by size.  A workgroup of the smallest tile reads x and W anew for
// every 16 x 16 outputs but has the most loads in flight, so it serves calls of
// one row tile and, by the number of chunks, of up to `small` tiles: the fewer
// chunks a workgroup has, the more of them share a CU.  Above, 2 x 2 tiles, and
// from six chunks on, past four tiles per CU, 2 x 4, which fill the LDS of a CU:
// these want their 192 workgroups, and a second round of them that an odd row
// tile pads or that only a few fill costs more than small tiles do.  us on 1x1 /
// 2x2 / 2x4: 64 rows 1024 -> 1024 4.1 / 6.0 / 8.8, 2048 -> 2048 6.7 / 7.8 /
// 11.4, 2048 -> 50256 99 / 86 / 80; 32 rows 64 -> 8192 3.6 / 4.7 / 6.8, 256 ->
// 8192 4.4 / 5.6 / 7.6; 128 rows 256 -> 2048 3.7 / 4.8 / 7.1, 320 -> 8192 9.4 /
// 7.8 / 9.0, 1088 -> 4096 11.9 / 11.2 / 10.1, 1024 -> 50256 84 / 50 / 58; 96
// rows 1088 -> 3072 8.4 / 10.9 / 9.7, 2048 -> 6144 20.8 / 21.0 / 23.2; 48 rows
// 1088 -> 12000 14.6 / 17.2 / 19.7, 2048 -> 12000 22.5 / 23.6 / 25.0; 16 rows
// 1984 -> 12000 13.5 / 17.4 / 15.8.  9 to 16 chunks of 256 (K <= 4096) take 16
// waves with a chunk each (4096 -> 1024: 64 rows 7.3 on 1x1, 9.1 on 2x1; 128
// rows 11.8 and 9.1), longer reductions 8 waves that loop (8192 -> 2048 on 1x1 /
// 1x2: 32 rows 12.2 / 17.0, 64 rows 20.9 / 16.7).
constexpr FewKind few_kind(int M, int N, int K) {
  const long rt = ceil_div(M, 16), t = rt * ceil_div(N, 16);
  if (K > 4096) return t > 256 ? kFewLong1x2 : kFewLong1x1;
  if (K > 2048) return t > 256 && rt > 1 ? kFewDeep2x1 : kFewDeep1x1;
  const int nc = lin_chunks(K);
  const int small = nc == 1 ? 8192 : nc == 2 ? 2304 : nc <= 4 ? 1536 : nc == 5 ? 768 : 512;
  if (t <= small || rt == 1) return kFew1x1;
  if (nc <= 4 || t <= 1024) return kFew2x2;
  const long wide = ceil_div(rt, 2) * ceil_div(N, 64);
  const bool odd = rt % 2, spill = wide > 256 && (odd || wide <= 320);
  return wide < 192 || spill || (odd && nc == 5) ? kFew1x1 : kFew2x4;
}

// The maps with the LayerNorm in the same kernel: column tiles and waves per
// chunk of k_linear_few_ln, or, with waves 0, row and column tiles and weight
// steps in flight of k_linear_skinny_ln.
struct FewLnPlan {
  int rt, g, wpc, u;
};
constexpr FewLnPlan kFewLnPlans[] = {{1, 1, 1, 0}, {1, 2, 1, 0}, {1, 4, 1, 0}, {1, 2, 2, 0}, {1, 4, 2, 0},
                                     {1, 1, 0, 8}, {1, 2, 0, 8}, {2, 4, 0, 4}};
enum FewLnKind { kLn1x1, kLn1x2, kLn1x4, kLn1x2Two, kLn1x4Two, kLnFrag1x1, kLnFrag1x2, kLnFrag2x4 };
constexpr int few_ln_threads(const FewLnPlan& p, int K) { return 64 * lin_chunks(K) * (p.wpc ? p.wpc : 1); }
constexpr long few_ln_lds_bytes(const FewLnPlan& p, int K) {
  const long nc = lin_chunks(K);
  if (p.wpc) return nc * p.wpc * FewTile::BYTES + 1024 + nc * p.g * 1024;
  const long sums = nc * 1024 * p.rt * p.g, stats = 4L * K + 2 * nc * 16 * p.rt * 4;
  return sums > stats ? sums : stats;
}

// Column tiles per workgroup by the number t of 16 x 16 tiles: as many as leave
// about one workgroup per CU, since each normalizes its 16 rows anew, with two
// waves per chunk where a wave would otherwise wait for them alone (K <= 1024).
// Past four tiles per CU the weights' reads count for more, and the widest tile
// wins: four columns with one wave per chunk at K <= 1024, 32 rows x 64 columns
// on MFMA-fragment loads, which normalize half as often, at K > 1024 -- but not
// for a single row tile, half of which would be padding.  Rows of 64 or 128
// values fill a quarter or half of a 512-byte piece: there the fragment loads
// stay, one row tile each (64 rows 64 -> 512: 4.0 us on 16 x 16, 4.4 on 1x2).
// us on 1x1 / 1x2 / 1x4 tiles with one wave per chunk, 1x2 / 1x4 with two, 32 x
// 64 on fragments: 64 rows 1024 -> 1024 5.6 / 6.3 / 7.9, 5.7 / 7.3, 11.6; 1024
// -> 4096 10.2 / 8.5 / 8.3, 8.1 / 7.7, 11.6; 128 rows 1024 -> 4096 16.4 / 13.4 /
// 11.0, 12.6 / 13.0, 11.8; 16 rows 768 -> 50256 22.2 / 21.2 / 22.7, 22.2 / 25.8,
// 26.2; 1024 -> 50256 27.8 / 26.4 / 27.0, 25.2 / 31.8, 34.7; 2048 -> 2048 7.1 /
// 8.7 / 11.7, - , 16.2; 2048 -> 12000 20.6 / 21.3 / 18.7, - , 22.1; 64 rows 2048
// -> 3072 17.0 / 15.8 / 11.8, - , 17.5; 2048 -> 8192 40.9 / 33.2 / 25.2, - , 21.0.
constexpr FewLnKind few_ln_kind(int M, int N, int K) {
  const long rt = ceil_div(M, 16), t = rt * ceil_div(N, 16);
  if (K <= 128 && t <= 2048) return t <= 256 ? kLnFrag1x1 : kLnFrag1x2;
  if (K <= 512) return t <= 2048 ? kLn1x2Two : kLn1x4Two;
  if (t <= 256) return kLn1x1;
  if (K <= 1024) {
    if (t <= 512 || (t > 1024 && t <= 1536)) return kLn1x2Two;
    if (t <= 1024) return kLn1x4Two;
    return rt > 1 ? kLn1x4 : K > 768 ? kLn1x2Two : kLn1x2;
  }
  if (t <= 512) return kLn1x2;
  return t <= 1024 || rt == 1 ? kLn1x4 : kLnFrag2x4;
}

// ---------------------------------------------------------------- few rows by a very wide map

// The wide kernel serves fp32 maps of at most 64 rows with K a multiple of
// 256 up to 2048 whose x rows fit in LDS (16 row tiles of K + 8 bf16 each:
// 64 rows up to K = 1024, 32 rows at K = 2048) and at least 8192 columns.
constexpr int kWideLds = 160 * 1024;
constexpr int wide_lds(int rt, int k) { return rt * 16 * (k + 8) * 2; }
constexpr bool wide_fits(int M, int N, int K) {
  return M >= 1 && M <= 64 && K % 256 == 0 && K <= 2048 && N >= 8192 && wide_lds((M + 15) / 16, K) <= kWideLds;
}

// ---------------------------------------------------------------- many rows

template <int BM_, int BN_, int BK_, int NS_, int WAVES_M, int WAVES_N>
struct GemmCfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, NS = NS_;
  static constexpr int NW = WAVES_M * WAVES_N, NT = 64 * NW;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 16, TN = WN / 16;
  static constexpr int CPR = BK / 8;                 // 16-byte chunks per LDS row
  static constexpr int RPI = 1024 / (BK * 2);        // rows per DMA instruction (1 KiB)
  static constexpr int R256 = 256 / (BK * 2);        // rows per 256 bytes
  static constexpr int IA = BM / RPI / NW, IB = BN / RPI / NW;
  static constexpr int STAGE = (BM + BN) * BK;       // elements per stage
  static constexpr int PER_CU = NS * STAGE * 2 <= 80 * 1024 ? 2 : 1;   // workgroups that fit a CU's LDS
  static constexpr bool PLAIN = NS == 2;             // no operands fetched ahead of their stage
  static_assert(!PLAIN || PER_CU == 2, "the next tile's fill needs the pipelined loop's last barrier");
  static_assert(IA * RPI * NW == BM && IB * RPI * NW == BN, "DMA rows must tile the stage");
  static_assert(NS >= 2 && NS <= 5, "ring depth");
  static constexpr int swz(int r) { return (r / R256) % CPR; }
};

// The tiles of a many-row map.  A wide tile moves fewer bytes from L2 into
// LDS per product, a small one fills the 256 CUs on small outputs.
using GemmWide = GemmCfg<128, 256, 64, 3, 2, 4>;   // one workgroup of 8 waves per CU (144 KB of LDS)
using GemmTall = GemmCfg<128, 128, 64, 4, 2, 4>;   // one of 8 waves per CU (128 KB)
using GemmPair = GemmCfg<128, 128, 64, 2, 2, 2>;   // two of 4 waves per CU (64 KB each)
using GemmSmall = GemmCfg<64, 64, 64, 4, 2, 2>;    // two of 4 waves per CU (64 KB each)
using GemmBrief = GemmCfg<64, 64, 64, 2, 2, 2>;    // four of 4 waves per CU (32 KB each): short reductions
enum GemmTile { kGemmWide, kGemmTall, kGemmPair, kGemmSmall, kGemmBrief };

// The tile of an M x N x K map: the cheapest by rounds over the 256 CUs.  A
// round of a tile is priced by what its workgroups take when j of them share a
// CU, (step + step_more (j - 1)) per 64 columns of K plus base + base_more (j -
// 1) for their start and end, in hundredths of a us: over 1994 measured maps (M
// 129 .. 8192, N 64 .. 12001, K 64 .. 8192, every epilogue) the choice costs
// 0.3% over the best tile on average, and more than 5% in one of a hundred.  A
// wide tile moves the fewest bytes per product but starts slowest, so the price
// has to know K.  us on wide / tall / pair / small / brief tiles: 320 x 8192 x
// 320 10.5 / 7.5 / 7.9 / 7.5 / 6.5, 640 x 2048 x 512 13.5 / 9.3 / 10.7 / 6.8 /
// 7.5, 2048 x 3072 x 256 11.5 / 12.8 / 10.9 / 11.8 / 10.8, 1024 x 3072 x 768
// 16.2 / 11.3 / 12.8 / 12.6 / 10.7, 8192 x 2304 x 768 47.1 / 45.0 / 43.1 / 54.0
// / 49.8, 640 x 8192 x 4096 58 / 73 / 66 / 78 / 98, 8192 x 8192 x 2048 283 /
// 340 / 310 / 437 / 416.
struct GemmPrice {
  int bm, bn, per_cu, step, base, step_more, base_more;
};
constexpr GemmPrice kGemmPrice[] = {
    {128, 256, 1, 76, 625, 0, 0},    // wide
    {128, 128, 1, 47, 350, 0, 0},    // tall
    {128, 128, 2, 62, 298, 30, 223}, // pair
    {64, 64, 2, 22, 107, 14, 56},    // small
    {64, 64, 4, 32, 68, 13, 61},     // brief
};
constexpr GemmTile gemm_tile(int M, int N, int K) {
  int best = 0;
  long least = 0;
  for (int i = 0; i < 5; ++i) {
    const GemmPrice& p = kGemmPrice[i];
    const long tiles = (long)((M + p.bm - 1) / p.bm) * ((N + p.bn - 1) / p.bn);
    auto round = [&](long j) { return (p.step + p.step_more * (j - 1)) * (K / 64) + p.base + p.base_more * (j - 1); };
    const long full = tiles / (256 * p.per_cu), rest = tiles % (256 * p.per_cu);
    const long price = full * round(p.per_cu) + (rest ? round((rest + 255) / 256) : 0);
    if (i == 0 || price < least) {
      least = price;
      best = i;
    }
  }
  return (GemmTile)best;
}

// Order index -> tile of a tiles_m x tiles_n map (false: none there): each XCD
// takes a contiguous range, in groups of 8 row tiles.
struct GemmPlace {
  int tm, tn;
  bool ok;
};
constexpr GemmPlace gemm_place(int i, int tiles_m, int tiles_n) {
  const int T = tiles_m * tiles_n, pid = i < xcd_grid(T) ? xcd_order(i, T) : -1;
  if (pid < 0) return {0, 0, false};
  const int per_group = 8 * tiles_n, g0 = (pid / per_group) * 8, gsz = tiles_m - g0 < 8 ? tiles_m - g0 : 8;
  return {g0 + (pid % per_group) % gsz, (pid % per_group) / gsz, true};
}
// Workgroups of a launch: where one fills a CU, it takes order index i, i +
// grid, .. (the grid is a multiple of 8, so all of them on its XCD).
constexpr int gemm_grid(int per_cu, int T) { return per_cu == 1 && xcd_grid(T) > 256 ? 256 : xcd_grid(T); }

}  // namespace smem
