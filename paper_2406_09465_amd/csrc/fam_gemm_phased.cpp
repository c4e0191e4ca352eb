// Phased main loop of the GEMM, conv and split-K families: products and implicit
// convolutions of plain 16-bit or fp32 operands staged direct to LDS, one barrier
// per k-tile with the matrix cores busy across it, long contractions split over
// workgroups.
//
// What bounds it: of a 16384 x 1024 x 4096 product with 256 x 256 tiles (109 us,
// 1.26 PFLOP/s; the 128 x 128 tiles staged as before took 195 us) the loads
// alone took 101 us in a probe and the products with their LDS reads alone 72, so
// the tile is as large as registers and LDS allow and the loads run under the
// products; the L2 misses are the compulsory ones, and each compute unit's L1
// holds 40 to 61 requests of 340 to 390 clocks and refuses more 28 to 37 % of the
// time.  LDS reads cost nothing measurable: two wave rows of 128 tile rows each
// read the right operand, whose transposing reads are the slow ones, only twice.
//
// A k-tile is NP phases: its k-steps, and the wave's row blocks in pairs.  Phase
// p multiplies fragments that were read one or two phases before, and the barrier
// that hands a tile over stands before the LAST phases: by then every wave holds
// their fragments in registers, so the stage is free, the next loads are issued
// into it at once, and the last phases' MFMAs cover the barrier and the first
// fragment reads of the next tile.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "families.h"
#include "gemm_common.h"

namespace korch {

static thread_local bool g_workgroup_splits = true;
void set_workgroup_splits(bool on) { g_workgroup_splits = on; }
bool workgroup_splits() { return g_workgroup_splits; }

static bool env_set(const char* n) {
  const char* e = getenv(n);
  return e && *e;
}

// Splitting a tile's contraction over workgroups pays where tiles leave compute
// units idle and the chain of k-tiles is long (the second product of an MLP
// block on few rows): up to one workgroup per compute unit, sixteen parts and
// two k-tiles each.  128 x 768 x 3072: 6.0 us in four parts against 9.2 (12.4
// staged through registers); 16 x 1024 x 4096: 5.1 against 8.7; 49 x 960 x 2240
// in fp32 6.7 against 11.6.
static bool splits_fit(int bm, int bn, int64_t tiles, int ks, int kg, double kt) {
  return workgroup_splits() && tiles * ks <= 256 && kt >= 2.0 * ks * kg && (double)tiles * ks * bm * bn * 4 <= 16.0 * (1 << 20);
}
// The hand-off of a split (partial tiles out, a counter, the last workgroup's
// sum): per part, more the more workgroups write partial tiles at once (`fill`:
// workgroups per compute unit).
static double handoff(int bm, int bn, int ks, int kg, double fill, bool f32) {
  if (ks == 1) return 0.0;
  const double area = bm * bn / 2048.0;
  return 1.0 + 0.2 * area + ks * area * (f32 ? 0.06 + 0.055 * fill : 0.07 + 0.22 * fill) + (kg > 1 ? 0.4 : 0.0);
}

// Tile shape, waves, k-groups and stages of the phased path; false: not taken.
//
// Each shape's cost on a product is predicted from the k-tile (64) times it
// reached when the chip was full of it (measured on products of 128 to 16384
// rows, contractions of 128 to 4096): t1 us with one workgroup per compute
// unit, tc us with the c that fit there at once (their k-tiles together), and
// ov us per round of workgroups for the first loads and the epilogue.  The last,
// partial round pays for the workgroups it puts on one compute unit.  Large
// tiles draw the fewest operand bytes per product, which is what bounds a full
// chip (see above); small tiles with deep stages cover latency when there are few
// of them.
//
// What is not a full chip of cache-resident operands is priced by terms fitted
// to 2700 16-bit and 800 fp32 kernels (every shape, 1 to 16384 rows, 1 to 16
// parts; to about 12 % warm, 16 % after a cache flush): a k-tile takes 0.7 (fp32
// 0.83) of its full-chip time on an empty chip and all of it from 142 workgroups
// on; operands of 32 MB, which come past the L2s, take 1.3 times as long (which
// weighs against the hand-off of a split only); and
// every k-tile of a workgroup's chain waits 0.1 us (fp32 0.03) per 100 tile rows
// and columns longer when its operands are first touched and the chip is too
// empty to hide it, of which half counts (they are cold in one use, warm in
// another).  So short chains in many parts are taken over two k-groups or few
// parts: 25 x 64 x 1344, batch of 8: 3.8 us in 7 parts (5.2 after a flush), 4.3
// (7.4) in two k-groups; 28 x 120 x 57384: 15 (24) in 16 parts, 25 (43) in 8;
// 436 x 2976 x 5624: 29 (36) as 128 x 96 tiles in two parts, 38 (55) as 128 x 64.
// `reads_rows`: the epilogue reads tensors that differ from row to row.
static bool phased_tiles(GemmSpec& sp, bool reads_rows) {
  if (const char* e = getenv("KORCH_GEMM_PHASED")) {
    int bm, bn, wm, wn, kg, st, bk, ks = 1;
    if (sscanf(e, "%d,%d,%d,%d,%d,%d,%d,%d", &bm, &bn, &wm, &wn, &kg, &bk, &st, &ks) < 7) return false;
    if (bm < 16 || bm > 512 || bn < 16 || bn > 512 || wm < 1 || wm > 8 || wn < 1 || wn > 8 || kg < 1 || kg > 8 || bk < 16 || bk > 64 || st < 2 ||
        st > 12 || ks < 1 || ks > 256)
      return false;
    sp.BM = bm, sp.BN = bn, sp.WM = wm, sp.WN = wn, sp.KG = kg, sp.PST = st, sp.BK = bk, sp.KS = ks;
    return true;
  }
  struct Shape_ {
    int bm, bn, wm, wn, kg, st, c;
    double t1, tc, ov;
  };
  double best = 1e300;
  // A convolution whose channels end half a k-tile short has k-tiles of half the
  // size (plan_phased), of which a tile's left rows must still be a whole number
  // of 1 KiB blocks for every wave.
  auto stages = [&](const Shape_& h, int bk) {
    if (sp.conv && sp.Cin % bk) bk /= 2;
    return h.bm * bk * dtype_bytes(sp.mtype) % (1024 * h.wm * h.wn) == 0;
  };
  if (sp.mtype == KORCH_F32) {
    // fp32 products are bound by their MFMAs (16x16x4: a quarter of a 16-bit
    // k-step's products in twice the clocks), so what a tile costs is its area
    // and how evenly the tiles fall on the compute units: t1 us per k-tile (32)
    // when a compute unit has one tile (its waves wait alone), tc us per tile
    // when it has several, which also pay for their first loads and stores one
    // after another, more than in proportion to their area (`turn`; 4967 x 1688 x 32
    // with a residual: 32 x 64 tiles 14.4 us, 64 x 64 17.3, 64 x 128 19.2).  2048 x
    // 3072 x 768: 64 x 96 tiles 74.9 us (128 x 96 staged through registers 83.4);
    // 2048 x 768 x
    // 3072: 73.4 in two k-groups (92.5); 340 x 256 x 1024: 32 x 32 tiles 6.9 (64
    // x 64: 23.2).
    static const Shape_ f32s[] = {
        {64, 128, 2, 2, 1, 2, 0, 1.14, 0.97, 4.0},  {64, 96, 2, 2, 1, 2, 0, 0.80, 0.745, 3.5}, {64, 64, 2, 2, 1, 2, 0, 0.62, 0.475, 3.0},
        {32, 64, 2, 2, 1, 4, 0, 0.32, 0.25, 2.5},   {32, 32, 2, 2, 1, 4, 0, 0.172, 0.13, 1.8}, {64, 96, 2, 2, 2, 3, 0, 0.82, 0.82, 3.0},
        {32, 64, 2, 2, 2, 6, 0, 0.31, 0.31, 2.0},   {32, 32, 2, 2, 2, 6, 0, 0.165, 0.165, 1.6},
    };
    const double KT = (double)((sp.K + 31) / 32);
    for (const Shape_& h : f32s) {
      if (!stages(h, 32)) continue;
      const int64_t tiles = (sp.M + h.bm - 1) / h.bm * ((sp.N + h.bn - 1) / h.bn) * sp.batch, n = (tiles + 255) / 256;
      // (over many tiles of a short contraction 32 x 32 ones read the operands too often where 64 columns are
      // not padding: 1687 x 872 x 48, batch of 8, 37.6 us after a flush, 32 x 64 34.1)
      if (n > 4 && KT <= 6 && h.bn == 32 && h.bm == 32 && sp.M > 32 && sp.N > 32) continue;
      const double area = h.bm * h.bn / 2048.0, turn = reads_rows ? 0.6 * area - 0.1 : 0.08 + 0.22 * area;
      for (int ks = 1; ks <= 16; ++ks) {
        if (ks > 1 && !splits_fit(h.bm, h.bn, tiles, ks, h.kg, KT)) break;
        const double kt = std::ceil(KT / ks), fill = std::min(1.0, tiles * ks / 256.0);
        if (h.kg > 1 && (n > 1 || kt < 8)) continue;  // two k-groups share the compute unit of one tile
        const double cost = h.ov + (n - 1) * turn + kt * (n == 1 ? h.t1 * (0.83 + 0.17 * fill) : n * h.tc) +
                            handoff(h.bm, h.bn, ks, h.kg, fill, true) + 0.00016 * kt * (h.bm + h.bn) * (1.0 - std::min(1.0, 1.8 * fill));
        if (cost < best) {
          best = cost;
          // (more tiles of a short contraction than fit on a compute unit hide the loads
          // better than stages: 4967 x 1688 x 32 in 32 x 64 tiles 18.7 us with four, 14.4
          // with two)
          sp.BM = h.bm, sp.BN = h.bn, sp.WM = h.wm, sp.WN = h.wn, sp.KG = h.kg, sp.PST = n > 4 && KT <= 6 ? 2 : h.st, sp.BK = 32, sp.KS = ks;
        }
      }
    }
    if (sp.K % 32 && sp.K % 32 <= 16 && sp.K <= 112 && !sp.conv && sp.KS == 1 && sp.KG == 1 &&
        (sp.M + sp.BM - 1) / sp.BM * ((sp.N + sp.BN - 1) / sp.BN) * sp.batch > 4 * 256) {
      // a short contraction over many tiles: k-tiles of 16 (of 64 rows at least,
      // so that every wave stages a block) save the MFMAs of an empty half k-tile
      if (sp.BM == 32) sp.BM = sp.BN = 64;
      sp.BK = 16, sp.PST = (int)std::min<int64_t>(4, std::max<int64_t>(2, (sp.K + 15) / 16));
    }
    return true;
  }
  static const Shape_ shapes[] = {
      {256, 256, 2, 4, 1, 2, 1, 1.50, 1.50, 9.5}, {256, 128, 2, 4, 1, 3, 1, 0.87, 0.87, 4.9}, {128, 128, 2, 2, 1, 2, 2, 0.62, 1.00, 3.2},
      {128, 128, 2, 4, 1, 4, 1, 0.50, 0.50, 2.6}, {128, 96, 2, 2, 1, 2, 2, 0.60, 0.88, 2.8},  {128, 96, 4, 2, 1, 5, 1, 0.46, 0.46, 2.2},
      {128, 64, 4, 2, 1, 5, 1, 0.31, 0.31, 2.2},  {128, 64, 2, 2, 1, 3, 2, 0.31, 0.57, 2.4},  {64, 128, 2, 2, 1, 3, 2, 0.31, 0.56, 2.3},
      {64, 64, 2, 2, 1, 4, 2, 0.245, 0.38, 1.7},   {32, 64, 2, 2, 1, 6, 2, 0.17, 0.29, 1.6},   {32, 64, 2, 2, 2, 6, 1, 0.165, 0.165, 1.6},
  };
  const double KT = (double)((sp.K + 63) / 64);
  if (KT <= 2 && sp.N % 8) {
    // One or two k-tiles and output rows that take narrow stores: the stores are
    // the time, issued best by many small workgroups (1477 x 1477 x 128: 128 x 96
    // tiles 6.1 us, 64 x 128 7.1, 64 x 64 5.5; 2001 x 501 x 96: 64 x 64 4.4, 32 x 64 3.7).
    // One k-step of 32 has nothing to stage ahead (1477 x 1477 x 16: 4.2 us with
    // register staging, 4.7 here).
    if (sp.K <= 32) return false;
    sp.BM = (sp.M + 63) / 64 * ((sp.N + 63) / 64) * sp.batch <= 256 ? 32 : 64;
    sp.BN = 64, sp.WM = sp.WN = 2, sp.KG = 1, sp.PST = 2, sp.BK = 64, sp.KS = 1;
    return true;
  }
  const int64_t tiles64 = (sp.M + 63) / 64 * ((sp.N + 63) / 64) * sp.batch;
  const bool three = sp.K > 80 && sp.K <= 96;
  if ((KT <= 1 || three) && !sp.conv && tiles64 > 256) {
    // One k-tile over more than a round of tiles is all first loads and stores, and
    // so are three k-steps of 32, in k-tiles of one step that leave no quarter of a
    // second k-tile empty.  An epilogue that reads tensors of the output's shape
    // goes through the fp32 C tile, of which small tiles keep more per compute unit
    // (in us: 623 x 8000 x 64 64 x 64 tiles 5.6, 64 x 128 7.5, 128 x 128 7.0, staged
    // through registers 6.5; 196 x 3328 x 64, batch of 16: 10.6, 13.9, 12.7, 15.4; 134
    // x 7776 x 96, batch of 8: 10.4, 12.4, 15.5, 11.3).  The rest store as fast from
    // any tile, and wider ones read the operands fewer times (2206 x 5088 x 64 7.8,
    // 7.3, 8.2, 8.2; after a flush 11.8, 9.4, 10.2, 9.8; 20000 x 256 x 96 6.6, 6.4, 6.9,
    // 7.1), 128 x 128 fastest in one nearly full round of two per compute unit (6867
    // x 1024 x 64: 4.8 us in 432 tiles, 64 x 128 5.6).
    const int64_t t128 = (sp.M + 127) / 128 * ((sp.N + 127) / 128) * sp.batch, t64x128 = (sp.M + 63) / 64 * ((sp.N + 127) / 128) * sp.batch;
    sp.WM = sp.WN = 2, sp.KG = 1, sp.PST = three ? 3 : 2, sp.BK = three ? 32 : 64, sp.KS = 1;
    sp.BM = sp.BN = 64;
    if (!reads_rows && t128 > 384 && t128 <= 512) {
      sp.BM = sp.BN = 128;
    } else if (!reads_rows && t64x128 > 512 && (double)t64x128 * 2.0 <= 1.1 * (double)tiles64) {
      sp.BN = 128;
    }
    return true;
  }
  // operands past the L2s (a convolution's left operand is its image)
  const double left = sp.conv ? (double)sp.H * sp.W * sp.Cin : (double)sp.M * sp.K * sp.batch;
  const double bytes = 2.0 * (left + (double)sp.K * sp.N * sp.batch), far = 0.3 * std::min(1.0, bytes / 32e6);
  for (const Shape_& h : shapes) {
    // 96 columns do not divide the threads: a convolution's per-channel operands
    // would be loaded for every element (275 x 129, 64 to 256 channels, 1 x 1:
    // 13.9 us in 128 x 96 tiles, 11.6 in 128 x 128)
    if (h.bn == 96 && sp.conv) continue;
    // register relief 1: no 256 x 256 tiles (128 accumulators beside the loads of
    // an epilogue with three operands of the output's shape spill 17 registers;
    // 16384 x 4096 x 1024 with it takes 203 us in 256 x 128 tiles, 247 with
    // 128-row tiles staged through registers)
    if (h.bm * h.bn == 256 * 256 && reg_relief() >= 1) continue;
    if (!stages(h, 64)) continue;
    const int64_t tiles = (sp.M + h.bm - 1) / h.bm * ((sp.N + h.bn - 1) / h.bn) * sp.batch;
    for (int ks = 1; ks <= 16; ++ks) {
      if (ks > 1 && !splits_fit(h.bm, h.bn, tiles, ks, h.kg, KT)) break;
      const double kt = std::ceil(KT / ks), fill = std::min(1.0, tiles * ks / 256.0), busy = std::min(1.0, 1.8 * fill);
      // two k-groups (their loads share one compute unit): where it has one tile
      if (h.kg > 1 && (tiles * ks > 256 || kt < 8)) continue;
      const int64_t full = tiles * ks / (256 * h.c), rest = (tiles * ks - full * 256 * h.c + 255) / 256;
      double tr = h.c > 1 ? h.t1 + (h.tc - h.t1) * (double)(rest - 1) / (h.c - 1) : h.t1;
      if (full + rest == 1) tr *= 0.7 + 0.3 * busy;
      double body = (full * (kt * h.tc + h.ov) + (rest ? kt * tr + h.ov : 0.0)) * (1.0 + far);
      if (ks > 1) body = std::max(body, bytes / 5.2e6);  // no split makes the operands arrive faster than the memory's 5.2 TB/s
      const double cost = body + handoff(h.bm, h.bn, ks, h.kg, fill, false) + 0.0005 * kt * (h.bm + h.bn) * (1.0 - busy);
      if (cost < best) {
        best = cost;
        sp.BM = h.bm, sp.BN = h.bn, sp.WM = h.wm, sp.WN = h.wn, sp.KG = h.kg, sp.PST = h.st, sp.BK = 64, sp.KS = ks;
      }
    }
  }
  if (sp.K % 64 > 16 && sp.K % 64 <= 32 && sp.K <= 224 && !sp.conv && sp.KS == 1 && sp.BM == 128 && sp.PST == 2 &&
      (sp.BN == 128 || (sp.M + 127) / 128 * ((sp.N + 127) / 128) * sp.batch > 512)) {
    // A short contraction whose last k-tile of 64 is half empty, over more than a
    // round of 128-row tiles: k-tiles of 32, in three stages that still leave three
    // workgroups per compute unit (4780 x 4832 x 160: 19.0 us with k-tiles of 64,
    // 17.4 in four stages of 32, 15.6 in three; 1404 x 3320 x 224, batch of 8: 33.8,
    // 30.7, 28.5; 3000 x 2000 x 288, above the line, 8.0 and 8.4).
    sp.BN = 128, sp.BK = 32, sp.PST = 3;
  }
  return true;
}

// Row blocks per band of the fp32 C tile (a divisor of FM): at most four
// 16-byte output vectors per thread and band, and two bands in LDS.
static int phased_band(const GemmSpec& sp) {
  for (int f : {4, 2})
    if (sp.FM % f == 0 && sp.WM * 16 * f * sp.BN <= 64 / dtype_bytes(sp.mtype) * sp.NT && (size_t)2 * sp.WM * 16 * f * sp.LDC * 4 <= 160 * 1024) return f;
  return 1;
}

static size_t phased_smem(const GemmSpec& sp) {
  const size_t st = (size_t)sp.PST * sp.KG * (sp.BM + sp.BN) * sp.BK * dtype_bytes(sp.mtype);
  if (sp.acc_t) return std::max(st, (size_t)sp.OSB);
  return std::max(st, sp.KG > 1 ? (size_t)sp.BM * sp.LDC * 4 : (size_t)2 * sp.WM * 16 * phased_band(sp) * sp.LDC * 4);
}

// The stored tensor whose last two dimensions the kernel transposes to form the
// right operand (attention's keys), or -1.
static int transposed_source(const KInfo& ki, const GemmSpec& sp) {
  const Node& n = ki.g.nodes[sp.Bs[0]];
  const int r = (int)n.shape.size();
  if (n.op != KORCH_TRANSPOSE || r < 2 || ki.in.count(n.in[0]) || sp.pro.size() != 1) return -1;
  for (int d = 0; d + 2 < r; ++d)
    if (n.attrs.perm[d] != d) return -1;
  if (n.attrs.perm[r - 2] != r - 1 || n.attrs.perm[r - 1] != r - 2) return -1;
  for (int o : ki.k.outs)
    if (o == sp.Bs[0]) return -1;
  return n.in[0];
}

// Whether the epilogue reads a tensor that differs from row to row of the product.
static bool epilogue_reads_rows(const KInfo& ki, const GemmSpec& sp) {
  const Graph& g = ki.g;
  for (int v : sp.epi)
    for (int u : g.nodes[v].in) {
      if (sp.epi.count(u) || std::count(sp.mms.begin(), sp.mms.end(), u)) continue;
      const Shape& s = g.nodes[u].shape;
      if (s.size() >= 2 && s[s.size() - 2] != 1) return true;
    }
  return false;
}

// The first k-tile whose lines are touched ahead (those before are loaded by the
// time a touch is back), and the cache lines from there on.
constexpr int kTouchFrom = 16;
static int64_t touch_lines(const GemmSpec& sp) {
  return ((sp.K - (int64_t)kTouchFrom * sp.BK) * sp.N * dtype_bytes(sp.mtype) + 127) / 128;
}

bool plan_phased(const KInfo& ki, GemmSpec& sp, bool split_halves) {
  sp.KG = 0;
  // the switches of the older staging paths ask for those paths
  for (const char* n : {"KORCH_GEMM_CFG", "KORCH_GEMM_NS", "KORCH_GEMM_NO_KSPLIT", "KORCH_GEMM_DMA", "KORCH_GEMM_DMA8",
                        "KORCH_GEMM_DMA_KSPLIT", "KORCH_GEMM_DMA_2STAGE", "KORCH_GEMM_DMA_A3", "KORCH_GEMM_DMA_STAGES",
                        "KORCH_GEMM_SPLIT_STEPS", "KORCH_GEMM_SCHED", "KORCH_GEMM_FULL_CTILE", "KORCH_LDS_BANK_SHIFT"})
    if (env_set(n)) return false;
  if (reg_relief() >= 2) return false;
  if (sp.lnf || sp.mms.size() != 1 || sp.Bs.size() != 1 || !sp.side.empty() || !sp.rowred.empty()) return false;
  const int eb = dtype_bytes(sp.mtype), CE = 16 / eb;
  if (ki.in.count(sp.A)) return false;  // operands computed in the kernel
  const int bt = ki.in.count(sp.Bs[0]) ? transposed_source(ki, sp) : -1;
  if (ki.in.count(sp.Bs[0]) && bt < 0) return false;
  // rows start on whole dwords (what a load to LDS needs; 16 bytes are read from any)
  if (sp.conv) {
    // implicit GEMM: a k-tile lies within one filter tap, so its left rows are
    // pixels at one shift (weights [KH, KW, Cin, Cout] are a [K, N] matrix)
    if (bt >= 0 || sp.nb || sp.Cin % (4 * CE) || (double)sp.H * sp.W * sp.Cin * eb >= 2147483648.0) return false;
  }
  if (sp.K * eb % 4 || (bt < 0 && sp.N * eb % 4)) return false;
  // buffer loads: byte offsets below 2 GiB from a batch's operand
  if ((double)sp.M * sp.K * eb >= 2147483648.0 || (double)sp.K * sp.N * eb >= 2147483648.0) return false;
  // Products for which the older rule takes 192-wide tiles keep them and their
  // staging: three stages direct to LDS where the tiles divide the problem (4096 x
  // 3072 x 768 with a GELU: 22.9 us, phased 22.4), through registers elsewhere
  // (4095 rows, say).  That line is the older rule's, not one of cost; both sides
  // are measured at that one product only.
  if (!getenv("KORCH_GEMM_PHASED") && sp.BN == 192 && !sp.conv) return false;
  // So do small products of up to four k-tiles whose tiles divide them: there is
  // nothing to pipeline (1024 x 768 x 256: 3.8 us, phased 3.9; 16384 x 64 x 256:
  // 3.7 either way; 4096 x 1024 x 256, above the line: 6.7 and 6.0).
  if (!getenv("KORCH_GEMM_PHASED") && !sp.conv && sp.M * sp.N * sp.batch <= 1 << 20 && sp.K <= 256 && sp.K % 64 == 0 && sp.M % sp.BM == 0 &&
      sp.N % sp.BN == 0)
    return false;
  // Outputs of a few columns waste most of the narrowest tile: over more rows than
  // a round of 128-row tiles, those of a short contraction keep their own
  // tiles of 16 or 32 columns (5591 x 16 x 104, batch of 16: 5.7 us, phased 6.7 at
  // best; 5616 x 16 x 304, batch of 8: 4.8 and 6.0; 8006 x 32 x 40, batch of 16: 5.6
  // and 8.2; 5538 x 6 x 184, batch of 16: 7.6 and 18.4; above the line 72891 x 24 x
  // 72 7.2 and 5.4, 15161 x 12 x 600, batch of 8, 28.2 and 25.4; rows of 8 but not of
  // 16 bytes, which those tiles gather: 60667 x 4 x 436, batch of 2, 44.0 and 20.0; fp32 82312 x 8 x 68 6.8 and 8.4, 16538 x 16 x 432, batch of 2,
  // 17.2 and 14.0).
  if (!getenv("KORCH_GEMM_PHASED") && !sp.conv) {
    const int64_t rows = sp.M * sp.batch;
    if (CE == 8 && sp.N <= 32 && rows > 128 * 256 && sp.K <= (sp.N % 4 == 2 || (sp.N <= 16 && sp.N % 8 == 0) ? 448 : 64)) return false;
    if (CE == 4 && sp.N <= 16 && rows > 65536 && sp.K <= 256) return false;
    // So do large outputs of one k-step, which are all stores and have nothing to
    // stage ahead (7613 x 6872 x 32: 22.9 us, 32.5 after a flush, phased 23.8 and
    // 43.8; 288 x 992 x 16, batch of 16: 4.3 and 5.2; below the line 1511 x 2656 x
    // 32 with a residual 6.1 and 4.2; fp32 186 x 5720 x 16, batch of 16: 15.1 and 21.1).
    if (sp.K <= (CE == 8 ? 32 : 16) && rows * sp.N >= 1 << 22) return false;
  }
  // Outputs of 16 columns waste most of the narrowest tile: a short convolution
  // to them keeps its own (300 x 300, 256 to 16 channels: 10.9 us, phased 12.6;
  // 141 x 141 with 3 x 3 taps of 128 channels, above the line: 9.5 and 8.9), as
  // does a long one over more than a round of its 64-row tiles (294 x 111, 3 x 3,
  // 512 to 16: 23.1 and 27.9; 141 x 140, 5 x 5, 96 to 16: 17.6 and 20.2; 290 x 98, 5 x
  // 5, 64 to 16, below the line: 11.4 and 10.2).
  if (!getenv("KORCH_GEMM_PHASED") && sp.conv && sp.N <= 16 && (sp.K <= 256 || (CE == 8 && sp.M > 64 * 256 && sp.K > 2048))) return false;
  // So does one over many pixels whose three or four k-tiles are of 32 channels
  // (275 x 129, 96 to 256 channels, 1 x 1: 11.0 us, phased 12.4).
  if (!getenv("KORCH_GEMM_PHASED") && sp.conv && CE == 8 && sp.Cin % 64 && sp.K <= 128 && sp.M * sp.N >= 1 << 22) return false;
  // fp32 outputs stored float by float after one k-tile: the stores are the time
  // (1477 x 1477 x 16: 4.7 us, phased 6.8; with K = 96, 1799 x 1799: 15.4 and 13.0).
  if (!getenv("KORCH_GEMM_PHASED") && CE == 4 && sp.N % 4 && sp.K <= 32) return false;
  GemmSpec t = sp;
  t.bt = bt;
  if (!phased_tiles(t, epilogue_reads_rows(ki, t))) return false;
  if (t.conv && t.Cin % t.BK) t.BK /= 2, t.PST = std::min(12, 2 * t.PST);  // the same LDS in twice the stages
  if (t.KS * t.KG > (t.K + t.BK - 1) / t.BK) t.KS = 1;
  // (partial tiles are addressed with 32-bit byte offsets)
  if ((double)((t.M + t.BM - 1) / t.BM * ((t.N + t.BN - 1) / t.BN) * t.batch) * t.KS * t.BM * t.BN * 4 >= 2147483648.0) t.KS = 1;
  // no stages that the contraction does not fill: short ones are bound by their
  // first loads and stores, which more workgroups per compute unit overlap
  if (!getenv("KORCH_GEMM_PHASED"))
    t.PST = (int)std::max<int64_t>(2, std::min<int64_t>(t.PST, ((t.K + t.BK - 1) / t.BK + t.KS * t.KG - 1) / (t.KS * t.KG)));
  // A long contraction whose 128-row tiles leave at most one per compute unit
  // is summed in two halves that are added at the end, as its k-split kernel
  // with register staging does: the results are the same to the bit (wave tiles
  // of up to 16 blocks, which leave registers for the second set of sums).
  t.KSEQ = t.KG == 1 && t.KS == 1 && split_halves && t.BM / t.WM * (t.BN / t.WN) <= 16 * 256 ? 2 : 1;
  if (t.BM % (16 * t.WM) || t.BN % (16 * t.WN)) return false;
  const int gw = t.WM * t.WN;  // waves per group
  t.NT = 64 * gw * t.KG;
  if (t.NT != 256 && t.NT != 512) return false;
  if (t.BK != 4 * CE && t.BK != 8 * CE) return false;  // rows of 64 or 128 bytes
  if ((t.BM * t.BK / (64 * CE)) % gw || t.BN * t.BK % (64 * CE)) return false;  // whole blocks, the left operand's shared evenly
  t.WTM = t.BM / t.WM, t.WTN = t.BN / t.WN;
  t.FM = t.WTM / 16, t.FN = t.WTN / 16;
  t.LDC = t.BN + 4;
  if (CE == 8 && bt < 0 && !dma_b_swizzle(t.BN / 8, t.dx0, t.dx1, t.dx3)) return false;
  t.acc_t = false;
  t.OSP = t.OSB = 0;
  t.CROWS = 0;
  if (t.KG == 1 && reg_epilogue_output(ki, t) >= 0) {
    t.acc_t = true;
    t.OSP = t.BN + 8;
    t.OSB = t.BM * t.OSP * 2;
  }
  if (phased_smem(t) + (t.KS > 1 ? 16 : 0) > 160 * 1024) return false;
  // Every workgroup of a long contraction meets the weights' next k-tile at the
  // same time, and after a flush each waits for HBM: the MLP block's second
  // product (4096 x 768 x 3072) took 29.1 us against 24.4 warm, the k-split
  // kernel before it 28.4.  So the workgroups first touch the later k-tiles
  // together, each a share of their cache lines: 25.6 us (the block 54.8 after a
  // flush, 58.5 without; 49.3 warm either way).  Fewer rows than this pay for the
  // touches when warm (1193 x 832 x 3328: the block 28.7 and 28.2 us, after a flush
  // 34.3 and 36.5); fp32 products are too slow to wait for HBM.
  t.touch = 0;
  if (CE == 8 && !t.conv && t.batch == 1 && t.KS == 1 && t.KG == 1 && t.M >= 2560 && t.K >= 2 * kTouchFrom * t.BK) {
    const int64_t wgs = (t.M + t.BM - 1) / t.BM * ((t.N + t.BN - 1) / t.BN), per = (touch_lines(t) + wgs - 1) / wgs;
    if (wgs >= 128 && wgs <= 512 && per <= t.NT) t.touch = (int)per;
  }
  sp = t;
  return true;
}


// Chunk of right row `k` that position `p` holds (load), or position of chunk
// `p` (read).  16-bit rows: p ^ f(k).  fp32 rows turn by four chunks per four
// rows: the four rows a fragment read takes at once (4 g + s, g = 0 .. 3) then
// start on different 64-byte parts of the banks.
static std::string b_chunk(const GemmSpec& sp, const std::string& p, const std::string& k, bool load) {
  if (sp.mtype != KORCH_F32) return "((" + p + ") ^ " + dma_fk(sp, k) + ")";
  const int P = sp.BN / 4;
  const std::string rot = "(4 * (((" + k + ") >> 2) & 3)) % " + std::to_string(P);
  return "(((" + p + ") + " + (load ? std::to_string(P) + " - " + rot : rot) + ") % " + std::to_string(P) + ")";
}

// Operand loads.  A block is 1 KiB: of the left operand 8 rows of 64 k, row r's
// 16-byte chunk c at position c ^ (r & 7) (k-tiles of 32: 16 rows, c ^ 2 (r / 4
// mod 2)), so that the lanes of a fragment read that the LDS serves together
// fall on 16 distinct bank groups; of the right operand 64 consecutive chunks of
// the [k][BN] tile, row k's chunk c at c ^ f(k) (dma_b_swizzle).
// Buffer loads, so rows and columns past the problem are clamped to its last
// ones (their products are never stored) and, where 64 does not divide K, the
// last k-tile's missing chunks read zero (an offset past the buffer).  M0 holds
// the LDS address; the wait state between its write and the load that reads it
// is spelled out, since the compiler does not see into the statement.
static std::string phased_loader(const KInfo& ki, const GemmSpec& sp, const std::map<int, int>& slot) {
  const std::string T = ctype(sp.mtype);
  const int eb = dtype_bytes(sp.mtype), CE = 16 / eb;  // element bytes, elements per chunk
  const int GW = sp.WM * sp.WN, PA = sp.BM * sp.BK / (64 * CE) / GW, NB = sp.BN * sp.BK / (64 * CE), PB = (NB + GW - 1) / GW;
  const int P = sp.BN / CE;                                                    // chunks per right row
  const int64_t SAB = (int64_t)sp.BM * sp.BK * eb, SBB = (int64_t)sp.BN * sp.BK * eb;  // bytes of a stage
  const int64_t KT = (sp.K + sp.BK - 1) / sp.BK;
  const int CR = sp.BK / CE, RB = 64 / CR;  // chunks per left row, rows per block
  std::ostringstream s;
  s << "  const int wv_ = __builtin_amdgcn_readfirstlane(wave);\n";
  s << "  const unsigned lds0_ = (unsigned)(size_t)(__attribute__((address_space(3))) void*)gsm_;\n";
  s << "  typedef int i32x4_ __attribute__((ext_vector_type(4)));\n";
  auto rsrc = [&](const char* X, int node, int64_t bytes) {
    s << "  const size_t p" << X << "_ = (size_t)((const " << T << "*)a.p[" << slot.at(node) << "] + ("
      << (sp.conv ? std::string("0") : operand_batch_offset(ki, sp, node)) << "));\n";
    s << "  const i32x4_ rs" << X << "_ = {__builtin_amdgcn_readfirstlane((int)(unsigned)p" << X
      << "_), __builtin_amdgcn_readfirstlane((int)((p" << X << "_ >> 32) & 0xffff)), " << (long long)bytes << ", 0x00020000};\n";
  };
  rsrc("A", sp.A, (sp.conv ? sp.H * sp.W * sp.Cin : sp.M * sp.K) * eb);
  rsrc("B", sp.bt >= 0 ? sp.bt : sp.Bs[0], sp.K * sp.N * eb);
  // k of this lane's left chunk within a tile (its position holds chunk c ^ g(row))
  s << "  const int lk_ = " << (CR == 8 ? "((l & 7) ^ (l >> 3)) * " : "((l & 3) ^ ((l >> 3) & 2)) * ") << CE << ";\n";
  s << "  unsigned va_[" << PA << "], vb_[" << PB << "];  // byte offsets of this lane's chunks at k-tile 0\n";
  if (sp.conv) s << "  int py_[" << PA << "], px_[" << PA << "];  // input pixel under the filter's first tap\n";
  s << "#pragma unroll\n  for (int i = 0; i < " << PA << "; ++i) {\n";
  s << "    i64 r = m0 + " << RB << " * (wv_ + i * " << GW << ") + l / " << CR << ";\n";
  if (sp.M % sp.BM) s << "    r = r < " << sp.M << "LL ? r : " << sp.M - 1 << "LL;\n";
  if (sp.conv)
    s << "    py_[i] = (int)r / " << sp.Wo << " * " << sp.stride << " - " << sp.pad << ";\n    px_[i] = (int)r % " << sp.Wo << " * " << sp.stride
      << " - " << sp.pad << ";\n    va_[i] = (unsigned)(((py_[i] * " << sp.W << " + px_[i]) * " << sp.Cin << " + lk_) * " << eb << ");\n  }\n";
  else
    s << "    va_[i] = (unsigned)((r * " << sp.K << "LL + lk_) * " << eb << ");\n  }\n";

  s << "#pragma unroll\n  for (int i = 0; i < " << PB << "; ++i) {\n";
  if (sp.bt >= 0) {
    s << "    i64 r = n0 + " << RB << " * (wv_ + i * " << GW << ") + l / " << CR << ";\n";
    if (sp.N % sp.BN) s << "    r = r < " << sp.N << "LL ? r : " << sp.N - 1 << "LL;\n";
    s << "    vb_[i] = (unsigned)((r * " << sp.K << "LL + lk_) * " << eb << ");\n  }\n";
  } else {
  s << "    const int q = (wv_ + i * " << GW << ") * 64 + l, k = q / " << P << ", p = q % " << P << ";\n";
  s << "    i64 c = n0 + " << b_chunk(sp, "p", "k", true) << " * " << CE << ";\n";
  if (sp.N % sp.BN) s << "    c = c < " << sp.N << "LL ? c : " << sp.N - CE << "LL;\n";
  s << "    vb_[i] = (unsigned)(((i64)k * " << sp.N << "LL + c) * " << eb << ");\n  }\n";
  }
  auto ld = [&](const char* off, const char* rs) {
    return std::string("      asm volatile(\"s_mov_b32 m0, %1\\n\\ts_nop 0\\n\\tbuffer_load_dwordx4 %0, %2, %3 offen lds\" :: \"v\"(") +
           off + "), \"s\"(la), \"s\"(" + rs + "), \"s\"(so) : \"memory\", \"m0\");\n";
  };
  const bool tail = sp.K % sp.BK != 0;
  // tile kt into stage st
  s << "  auto load_ = [&](const int kt, const int st) {\n";
  if (sp.conv) {
    // the tile's tap (ky, kx) and channels: a uniform shift of every pixel; taps
    // outside the image read zero (an offset past the buffer)
    s << "    const int tap_ = kt * " << sp.BK << " / " << sp.Cin << ", ky_ = tap_ / " << sp.KW << ", kx_ = tap_ % " << sp.KW << ";\n";
    s << "    const unsigned to_ = (unsigned)(((ky_ * " << sp.W << " + kx_) * " << sp.Cin << " + kt * " << sp.BK << " % " << sp.Cin << ") * "
      << eb << ");\n";
  }
  s << "    {\n    const unsigned so = __builtin_amdgcn_readfirstlane(" << (sp.conv ? "0u * " : "") << "(unsigned)kt * " << sp.BK * eb << "u);\n#pragma unroll\n    for (int i = 0; i < " << PA << "; ++i) {\n";
  s << "      const unsigned la = lds0_ + (unsigned)(st * " << SAB << " + (wv_ + i * " << GW << ") * 1024);\n";
  if (sp.conv)
    s << "      const unsigned vo = (unsigned)(py_[i] + ky_) < " << sp.H << "u && (unsigned)(px_[i] + kx_) < " << sp.W
      << "u ? va_[i] + to_ : 0x80000000u;\n"
      << ld("vo", "rsA_");
  else if (tail)
    s << "      const unsigned vo = kt == " << KT - 1 << " && lk_ >= " << sp.K % sp.BK
      << " ? 0x80000000u : va_[i];\n"
      << ld("vo", "rsA_");
  else
    s << ld("va_[i]", "rsA_");
  s << "    }\n    }\n";
  s << "    {\n    const unsigned so = __builtin_amdgcn_readfirstlane((unsigned)kt * " << eb * sp.BK * (sp.bt >= 0 ? 1 : sp.N) << "u);\n#pragma unroll\n    for (int i = 0; i < " << PB << "; ++i) {\n";
  if (NB % GW) s << "      if (i == " << PB - 1 << " && wv_ >= " << NB % GW << ") break;  // the first waves load one block more\n";
  s << "      const unsigned la = lds0_ + (unsigned)(" << sp.PST * SAB << " + st * " << SBB << " + (wv_ + i * " << GW << ") * 1024);\n";
  if (tail && sp.bt >= 0)
    s << "      const unsigned vo = kt == " << KT - 1 << " && lk_ >= " << sp.K % sp.BK << " ? 0x80000000u : vb_[i];\n" << ld("vo", "rsB_");
  else if (tail)
    s << "      const unsigned vo = kt == " << KT - 1 << " && ((wv_ + i * " << GW << ") * 64 + l) / " << P << " >= " << sp.K % sp.BK
      << " ? 0x80000000u : vb_[i];\n"
      << ld("vo", "rsB_");
  else
    s << ld("vb_[i]", "rsB_");
  s << "    }\n    }\n  };\n";
  return s.str();
}

static std::string phased_mainloop(const GemmSpec& sp, int64_t KTG, bool exact) {
  std::ostringstream s;
  const int64_t KT = (sp.K + sp.BK - 1) / sp.BK;
  const std::string T = ctype(sp.mtype), V8 = sp.mtype == KORCH_F32 ? "f32x4" : sp.mtype == KORCH_F16 ? "f16x8" : "bf16x8";
  const bool f32 = sp.mtype == KORCH_F32;
  const int eb = dtype_bytes(sp.mtype), CE = 16 / eb, KW = 4 * CE;  // k of one fragment read (four chunks)
  const std::string fn = sp.mtype == KORCH_F16 ? "__builtin_amdgcn_mfma_f32_16x16x32_f16"
                                               : "__builtin_amdgcn_mfma_f32_16x16x32_bf16";
  const int FH = sp.FM % 2 ? 1 : 2, H = sp.FM / FH, nkk = sp.BK / KW, NP = nkk * H;  // row blocks per phase; phases
  const int L = std::min(2, H), NA = 2 * L;  // phases a left fragment is read ahead; register sets
  const int NST = sp.PST, GW = sp.WM * sp.WN, PL = (sp.BM + sp.BN) * sp.BK / (64 * CE) / GW;  // loads per wave and tile
  const int PX = (sp.BN * sp.BK / (64 * CE)) % GW;  // waves with one load more
  // tiles per round: stages, left register sets and right register sets repeat
  int U = NST;
  while ((U * NP) % NA || (U * nkk) % 2) U += NST;
  // all stages of the left operand, then all of the right one: with 64 KiB or
  // less of each, a fragment's address is a lane's base plus an immediate
  const int64_t SAE = (int64_t)sp.BM * sp.BK, SBE = (int64_t)sp.BN * sp.BK;
  s << "  f32x4 acc[" << sp.FM << "][" << sp.FN << "];\n";
  s << "#pragma unroll\n  for (int i = 0; i < " << sp.FM << "; ++i)\n#pragma unroll\n  for (int j = 0; j < " << sp.FN
    << "; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};\n";
  s << "  " << V8 << " fa_[" << NA << "][" << FH << "], fb_[2][" << sp.FN << "];\n";
  s << "  const " << T << "* Af_ = (const " << T << "*)gsm_ + (wm * " << sp.WTM << " + (l & 15)) * " << sp.BK << ";\n";
  s << "  const int ca_ = " << (sp.BK / CE == 8 ? "((l >> 4) ^ (l & 7)) * " : "((l >> 4) ^ ((l >> 1) & 2)) * ") << CE << ";\n";
  if (sp.bt >= 0) {
    // rows of the right tile as the left one's
    s << "  const " << T << "* Bf_ = (const " << T << "*)gsm_ + " << NST * SAE << " + (wn * " << sp.WTN << " + (l & 15)) * " << sp.BK << ";\n";
  } else {
  s << "  const " << T << "* Bf_ = (const " << T << "*)gsm_ + " << NST * SAE << " + (" << (f32 ? "(l >> 4) * 4" : "(l >> 4) * 8 + ((l & 15) >> 2)") << ") * " << sp.BN << ";\n";
  s << "  int cb_[" << sp.FN << "];\n#pragma unroll\n  for (int j = 0; j < " << sp.FN << "; ++j) {\n";
  if (f32)
    s << "    const int n_ = wn * " << sp.WTN << " + j * 16 + (l & 15), k_ = (l >> 4) * 4;\n";
  else
    s << "    const int n_ = wn * " << sp.WTN << " + j * 16 + 4 * (l & 3), k_ = (l >> 4) * 8 + ((l & 15) >> 2);\n";
  s << "    cb_[j] = " << b_chunk(sp, "n_ / " + std::to_string(CE), "k_", false) << " * " << CE << " + n_ % " << CE << ";\n  }\n";
  }
  // left fragments of phase p (rows [p % H * FH, + FH), k-step p / H) of tile t
  // (counted within a round), right fragment j of its k-step kk
  auto setA = [&](int t, int p) { return ((t % U) * NP + p) % NA; };
  auto setB = [&](int t, int kk) { return ((t % U) * nkk + kk) % 2; };
  auto readA = [&](int t, int p) {
    std::ostringstream o;
    for (int i = 0; i < FH; ++i)
      o << "    fa_[" << setA(t, p) << "][" << i << "] = *(const " << V8 << "*)(Af_ + "
        << (t % NST) * SAE + ((p % H) * FH + i) * 16 * sp.BK << " + (ca_ ^ " << (p / H) * 4 * CE << "));\n";
    return o.str();
  };
  auto readB = [&](int t, int kk, int j) {
    std::ostringstream o;
    if (sp.bt >= 0) {
      o << "    fb_[" << setB(t, kk) << "][" << j << "] = *(const " << V8 << "*)(Bf_ + " << (t % NST) * SBE + j * 16 * sp.BK << " + (ca_ ^ "
        << kk * 4 * CE << "));\n";
      return o.str();
    }
    if (f32) {
      // the contraction's order is free as long as both fragments agree: lane
      // group g holds the consecutive k 4 g .. 4 g + 3 of the window (one
      // 16-byte read of the left operand), and product s takes their s-th
      o << "    {\n      const float* b_ = Bf_ + " << (t % NST) * SBE + kk * KW * sp.BN << " + cb_[" << j << "];\n      fb_[" << setB(t, kk)
        << "][" << j << "] = f32x4{b_[0], b_[" << sp.BN << "], b_[" << 2 * sp.BN << "], b_[" << 3 * sp.BN << "]};\n    }\n";
      return o.str();
    }
    o << "    fb_[" << setB(t, kk) << "][" << j << "] = __builtin_bit_cast(" << V8 << ", lds_tr_k8(Bf_ + "
      << (t % NST) * SBE + kk * KW * sp.BN << " + cb_[" << j << "], " << sp.BN << "));\n";
    return o.str();
  };
  // right fragments [FN h / parts, FN (h + 1) / parts)
  auto readBs = [&](int t, int kk, int h, int parts) {
    std::string o;
    for (int j = sp.FN * h / parts; j < sp.FN * (h + 1) / parts; ++j) o += readB(t, kk, j);
    return o;
  };
  // waits until at most the loads of n tiles are in flight: a wave's loads to
  // LDS complete in issue order, also where some come from HBM, some from a
  // cache and some lie out of the buffer's range (a probe of such mixes read
  // 1.3e10 words after partial waits, all of them landed)
  auto wait = [&](int n) {
    auto w = [](int c) { return "asm volatile(\"s_waitcnt vmcnt(" + std::to_string(c) + ")\" ::: \"memory\");\n"; };
    if (!n || !PX) return "    " + w(n * PL);
    return "    if (wv_ < " + std::to_string(PX) + ") " + w(n * (PL + 1)) + "    else " + w(n * PL);
  };
  // Where rows end inside a chunk, the last k-tile's chunk goes on into the next
  // row: those elements are zeroed in LDS once the tile has landed (index
  // `last` of the last part; the others pass).  The barrier is every wave's.
  const int64_t last = exact ? KTG - 1 : std::max<int64_t>(0, KTG - 2);
  const bool ragged = sp.K % CE != 0;
  auto trim = [&](int t) {
    std::ostringstream o;
    const int64_t kr = sp.K % sp.BK;
    const int GT = 64 * GW;
    o << "    if (kt1 == " << KT << ") {\n";
    for (int op = 0; op < (sp.bt >= 0 ? 2 : 1); ++op) {
      const int rows = op ? sp.BN : sp.BM;
      o << "      for (int r_ = tid; r_ < " << rows << "; r_ += " << GT << ") {\n        " << T << "* z_ = (" << T << "*)gsm_ + "
        << (op ? NST * SAE + (t % NST) * SBE : (t % NST) * SAE) << " + r_ * " << sp.BK << " + (" << kr / CE << " ^ "
        << (sp.BK / CE == 8 ? "(r_ & 7)" : "((r_ >> 1) & 2)") << ") * " << CE << ";\n#pragma unroll\n        for (int e = " << kr % CE
        << "; e < " << CE << "; ++e) z_[e] = (" << T << ")0.0f;\n      }\n";
    }
    o << "    }\n    __syncthreads();\n";
    return o.str();
  };
  // Tile j of the group, number t of a round.  `more`: tile j + NST exists (1)
  // or may exist (2); `next`: tile j + 1 exists; `steady`: tiles j + 2 .. j +
  // NST - 1 exist in every group and are the loads in flight beyond tile j + 1;
  // `live`: the group may have no tile j (a shorter last group).
  auto tile = [&](const std::string& j, int t, int more, bool next, bool steady, bool live, bool trims = false) {
    std::ostringstream o;
    for (int p = 0; p < NP; ++p) {
      if (p == NP - L && next) {
        // tile j + 1 has landed and every wave holds the rest of tile j
        o << wait(steady ? NST - 2 : 0) << "    __syncthreads();\n";
        if (trims) o << trim(t + 1);
        if (more)
          o << (more == 2 ? "    if (" + j + " + " + std::to_string(NST) + " < nkt_) " : std::string("    ")) << "load_(kt0 + " << j
            << " + " << NST << ", " << t % NST << ");\n";
      }
      const int q = p + L;
      if (q < NP) o << readA(t, q);
      else if (next) o << readA(t + 1, q - NP);
      for (int kk = 1; kk < nkk; ++kk)
        if (p / H == kk - 1) o << readBs(t, kk, p % H, H);
      if (p >= NP - L && next) o << readBs(t + 1, 0, p - (NP - L), L);
      o << (live ? "    if (" + j + " < nkt_) {\n" : "    {\n");
      const std::string A = "fa_[" + std::to_string(setA(t, p)) + "][i]", B = "fb_[" + std::to_string(setB(t, p / H)) + "][n]",
                        C = "acc[" + std::to_string((p % H) * FH) + " + i][n]";
      o << "#pragma unroll\n      for (int i = 0; i < " << FH << "; ++i)\n#pragma unroll\n        for (int n = 0; n < " << sp.FN << "; ++n) {\n";
      if (f32)
        for (int q = 0; q < 4; ++q)
          o << "          " << C << " = __builtin_amdgcn_mfma_f32_16x16x4f32(" << A << "[" << q << "], " << B << "[" << q << "], " << C
            << ", 0, 0, 0);\n";
      else
        o << "          " << C << " = " << fn << "(" << (sp.acc_t ? B + ", " + A : A + ", " + B) << ", " << C << ", 0, 0, 0);\n";
      o << "        }\n";
      o << "    }\n    __builtin_amdgcn_sched_barrier(0);\n";
    }
    if (sp.KSEQ > 1) {
      // the end of the first half: its sums are set aside
      o << "    if (" << j << " == " << (KTG + 1) / 2 - 1 << ") {\n#pragma unroll\n      for (int i = 0; i < " << sp.FM
        << "; ++i)\n#pragma unroll\n        for (int n = 0; n < " << sp.FN
        << "; ++n) { acc0_[i][n] = acc[i][n]; acc[i][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }\n    }\n";
    }
    return o.str();
  };
  if (sp.KSEQ > 1) s << "  f32x4 acc0_[" << sp.FM << "][" << sp.FN << "];  // the sums of the first half of the k-tiles\n";
  s << "  const int nkt_ = kt1 - kt0;\n  (void)nkt_;\n";
  const int64_t KS = exact ? KTG : KTG - 1;  // k-tiles that every group has
  for (int t = 0; t < NST && t < KTG; ++t)
    s << "  " << (t < KS ? "" : "if (" + std::to_string(t) + " < nkt_) ") << "load_(kt0 + " << t << ", " << t << ");\n";
  if (sp.touch)
    // (plan_phased; behind the loads of the first tiles, so that a wait for the
    // oldest loads does not wait for this one)
    s << "  unsigned touch_ = 0;\n  if (tid < " << sp.touch << " && (i64)wg * " << sp.touch << " + tid < " << touch_lines(sp)
      << "LL) touch_ = *(const unsigned*)((const char*)pB_ + " << (int64_t)kTouchFrom * sp.BK * sp.N * eb << "LL + ((i64)wg * " << sp.touch
      << " + tid) * 128);\n";
  // tile 0 landed; the tiles after it may be in flight
  s << wait(KS >= NST ? NST - 1 : 0) << "  __syncthreads();\n";
  if (ragged && last == 0) s << trim(0);
  for (int p = 0; p < L; ++p) s << readA(0, p);
  s << readBs(0, 0, 0, 1);
  // steady part: tile j + NST exists in every group, in rounds of U tiles
  const int64_t steady = KS > NST ? (KS - NST) / U * U : 0;
  if (steady > 0) {
    s << "#pragma unroll 1\n  for (int j = 0; j < " << steady << "; j += " << U << ") {\n";
    for (int u = 0; u < U; ++u) s << tile("(j + " + std::to_string(u) + ")", u, 1, true, true, false);
    s << "  }\n";
  }
  for (int64_t j = steady; j < KTG; ++j) {
    const int more = j + NST < KS ? 1 : j + NST < KTG ? 2 : 0;
    s << "  {\n" << tile(std::to_string(j), (int)(j % U), more, j + 1 < KTG, j + NST - 1 < KS, j >= KS, ragged && j + 1 == last)
      << "  }\n";
  }
  if (sp.KSEQ > 1)
    s << "#pragma unroll\n  for (int i = 0; i < " << sp.FM << "; ++i)\n#pragma unroll\n  for (int n = 0; n < " << sp.FN
      << "; ++n) acc[i][n] = acc0_[i][n] + acc[i][n];\n";
  if (sp.touch) s << "  asm volatile(\"\" :: \"v\"(touch_));\n";
  s << "  __syncthreads();\n";
  return s.str();
}

GenKernel gen_gemm_phased(const KInfo& ki, GemmSpec& sp, int index, const char* fam) {
  GenKernel gk;
  gk.family = KORCH_FAM_GEMM;
  gk.name = kernel_name(index, fam);
  std::map<int, int> slot;
  ki.assign_args(gk, slot);
  const int64_t ntn = (sp.N + sp.BN - 1) / sp.BN, ntm = (sp.M + sp.BM - 1) / sp.BM, KT = (sp.K + sp.BK - 1) / sp.BK;
  const int parts = sp.KG * sp.KS;  // of the k-tiles: the first KT % parts of them have one more
  const int64_t KTG = (KT + parts - 1) / parts;
  const int64_t tiles = ntn * ntm * sp.batch;
  // Split of the contraction over workgroups: every part's sums to scratch in
  // lane order (coherent stores), the tile's last workgroup adds them in part
  // order and runs the epilogue.  One counter per tile on a line of its own.
  const size_t part_bytes = (size_t)sp.BM * sp.BN * 4;
  int scr_slot = -1, cnt_slot = -1;
  gk.wg_split = sp.KS > 1;
  if (sp.KS > 1) {
    ArgRef scr;
    scr.kind = ArgRef::Scratch;
    scr.bytes = (size_t)tiles * sp.KS * part_bytes;
    scr_slot = (int)gk.args.size();
    gk.args.push_back(scr);
    ArgRef cnt;
    cnt.kind = ArgRef::Counter;
    cnt.bytes = (size_t)tiles * 128;
    cnt_slot = (int)gk.args.size();
    gk.args.push_back(cnt);
  }
  const std::string T = ctype(sp.mtype);
  const int GT = 64 * sp.WM * sp.WN;  // threads of a group
  std::ostringstream s;
  s << source_header((int)gk.args.size());
  s << "extern \"C\" __global__ void __launch_bounds__(" << sp.NT << ") __attribute__((amdgpu_waves_per_eu(2))) " << gk.name << "(KArgs a) {\n";
  s << "  __shared__ __attribute__((aligned(1024))) char smem[" << phased_smem(sp) << "];\n";
  if (sp.KG > 1) {
    s << "  const int kgrp = __builtin_amdgcn_readfirstlane(threadIdx.x / " << GT << ");  // which part of the k-tiles\n";
    s << "  char* gsm_ = smem + kgrp * " << sp.PST * (sp.BM + sp.BN) * sp.BK * dtype_bytes(sp.mtype) << ";  // this group's operand stages\n";
    s << "  const int tid = threadIdx.x % " << GT << ", l = tid & 63, wave = tid >> 6;\n";
  } else {
    s << "  char* gsm_ = smem;  // operand stages\n";
    s << "  const int tid = threadIdx.x, l = tid & 63, wave = tid >> 6;\n";
  }
  s << "  const int wm = wave / " << sp.WN << ", wn = wave % " << sp.WN << ";\n  (void)wm; (void)wn;\n";
  if (sp.KS > 1) s << "  const int split_ = blockIdx.x / " << tiles << ";  // which part of the k-tiles\n  __shared__ int last_;\n";
  s << gemm_tile_order(sp, ntm, ntn, sp.KS > 1 ? "blockIdx.x % " + std::to_string(tiles) : std::string("blockIdx.x"));
  if (parts > 1) {
    const std::string pt = sp.KS == 1 ? "kgrp" : sp.KG == 1 ? "split_" : "(split_ * " + std::to_string(sp.KG) + " + kgrp)", B_ = std::to_string(KT / parts), R_ = std::to_string(KT % parts);
    s << "  const int kt0 = " << pt << " * " << B_ << " + (" << pt << " < " << R_ << " ? " << pt << " : " << R_ << "), kt1 = kt0 + " << B_
      << " + (" << pt << " < " << R_ << " ? 1 : 0);\n";
  } else {
    s << "  const int kt0 = 0, kt1 = " << KT << ";\n";
  }
  s << phased_loader(ki, sp, slot);
  s << phased_mainloop(sp, KTG, KT % parts == 0);
  auto ctile = [&](const char* op) {
    std::ostringstream o;
    o << "#pragma unroll\n    for (int i = 0; i < " << sp.FM << "; ++i)\n#pragma unroll\n    for (int j = 0; j < " << sp.FN
      << "; ++j)\n#pragma unroll\n    for (int r = 0; r < 4; ++r) Cs[((" << (sp.KG > 1 ? "wm * " + std::to_string(sp.WTM) : std::string("0"))
      << ") + i * 16 + (l >> 4) * 4 + r) * " << sp.LDC << " + wn * " << sp.WTN << " + j * 16 + (l & 15)] " << op << " acc[i][j][r];\n";
    return o.str();
  };
  // The groups' sums one after another in group order into the fp32 C tile.
  auto groups = [&]() {
    std::string o;
    for (int q = 0; q < sp.KG; ++q) o += "  if (kgrp == " + std::to_string(q) + ") {\n" + ctile(q ? "+=" : "=") + "  }\n  __syncthreads();\n";
    return o;
  };
  if (sp.KS > 1) {
    // NV 16-byte vectors per thread: the accumulator blocks in lane order, or
    // (several k-groups, whose sums meet in the C tile first) the tile's rows
    const bool viaC = sp.KG > 1;
    const int VPR = sp.BN / 4, NV = viaC ? (sp.BM * VPR + sp.NT - 1) / sp.NT : sp.FM * sp.FN, LB = sp.NT * 16;
    const bool whole = !viaC || sp.BM * VPR % sp.NT == 0;
    const std::string TID = viaC ? "(int)threadIdx.x" : "tid";
    auto reg = [&](const std::string& i) {
      return viaC ? "*(f32x4*)(Cs + ((" + TID + " + " + i + " * " + std::to_string(sp.NT) + ") / " + std::to_string(VPR) + ") * " +
                        std::to_string(sp.LDC) + " + ((" + TID + " + " + i + " * " + std::to_string(sp.NT) + ") % " + std::to_string(VPR) + ") * 4)"
                  : "acc[" + i + " / " + std::to_string(sp.FN) + "][" + i + " % " + std::to_string(sp.FN) + "]";
    };
    const std::string in = whole ? "" : "if (" + TID + " + i * " + std::to_string(sp.NT) + " < " + std::to_string(sp.BM * VPR) + ") ";
    s << "  {\n";
    if (viaC) s << "  float* Cs = (float*)smem;\n" << groups();
    s << "  float* part_ = (float*)a.p[" << scr_slot << "];\n";
    s << "  const __amdgpu_buffer_rsrc_t rsP = __builtin_amdgcn_make_buffer_rsrc(part_, 0, " << tiles * sp.KS * part_bytes << ", 0x00020000);\n";
    s << "  const unsigned po_ = (unsigned)(wg * " << sp.KS << ") * " << part_bytes << "u + " << TID << " * 16;\n";
    s << "#pragma unroll\n  for (int i = 0; i < " << NV << "; ++i)\n    " << in << "coherent_store4(rsP, po_ + split_ * " << part_bytes
      << "u + i * " << LB << ", __builtin_bit_cast(float4, " << reg("i") << "));\n";
    s << "  __builtin_amdgcn_s_waitcnt(0);  // this wave's partial stores are performed\n  __syncthreads();\n";
    s << "  if (threadIdx.x == 0) {\n    int* cnt = (int*)a.p[" << cnt_slot << "] + wg * 32;\n";
    s << "    const int old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n";
    s << "    last_ = old == " << sp.KS - 1 << ";\n";
    s << "    if (last_) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);\n  }\n";
    s << "  __syncthreads();\n  if (!last_) return;\n";
    // up to 32 loads in flight per thread; past the tile or the last part they
    // repeat one that exists
    const int BS = std::max(1, std::min(sp.KS, 32 / NV));
    s << "  f32x4 sum_[" << NV << "];\n#pragma unroll\n  for (int i = 0; i < " << NV << "; ++i) sum_[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};\n";
    s << (sp.KS > BS ? "#pragma unroll 1\n" : "#pragma unroll\n") << "  for (int s0_ = 0; s0_ < " << sp.KS << "; s0_ += " << BS << ") {\n";
    s << "    f32x4 v_[" << BS << "][" << NV << "];\n";
    s << "#pragma unroll\n    for (int s_ = 0; s_ < " << BS << "; ++s_)\n#pragma unroll\n      for (int i = 0; i < " << NV
      << "; ++i) v_[s_][i] = __builtin_bit_cast(f32x4, coherent_load4(rsP, po_ + (s0_ + s_ < " << sp.KS << " ? s0_ + s_ : " << sp.KS - 1 << ") * "
      << part_bytes << "u + i * " << LB << "));\n";
    s << "#pragma unroll\n    for (int s_ = 0; s_ < " << BS << "; ++s_)\n#pragma unroll\n      for (int i = 0; i < " << NV << "; ++i)\n"
      << "        if (s0_ + s_ < " << sp.KS << ") sum_[i] += v_[s_][i];\n    }\n";
    s << "#pragma unroll\n  for (int i = 0; i < " << NV << "; ++i) " << in << reg("i") << " = sum_[i];\n";
    if (viaC) s << "  __syncthreads();\n";
    s << "  }\n";
  }
  // The epilogue's lane indices go through an opaque copy: its many LDS and
  // output addresses would otherwise be computed ahead of the main loop and
  // held (spilled) across it.
  s << "  int te_ = threadIdx.x;\n  asm volatile(\"\" : \"+v\"(te_));\n  {\n  const int tid = te_"
    << (sp.KG > 1 ? " % " + std::to_string(GT) : std::string()) << ", l = tid & 63, wave = tid >> 6, wm = wave / " << sp.WN
    << ", wn = wave % " << sp.WN << ";\n  (void)wm; (void)wn;\n";
  if (sp.acc_t) {
    s << gemm_reg_epilogue(ki, sp, slot, reg_epilogue_output(ki, sp));
  } else if (sp.KG > 1) {
    s << "  float* Cs = (float*)smem;\n" << (sp.KS == 1 ? groups() : std::string());
    s << "  {\n  const int tid = te_;\n";
    s << gemm_epilogue(ki, sp, slot, "ml * " + std::to_string(sp.LDC));
    s << "  }\n";
  } else {
    // The fp32 C tile in NQ bands, each FQ row blocks of every wave row, through
    // two LDS buffers: a band is evaluated and stored while the accumulators of
    // the later ones are still in registers, with one barrier per band.
    const int FQ = phased_band(sp), NQ = sp.FM / FQ, R = 16 * FQ, rows = sp.WM * R;
    s << "  float* Cs = (float*)smem;\n";
    std::string inv;  // loads that are the same for every element of a thread, once before the bands
    // one band's code, its row offsets left open (QROW_, QOFF_)
    const std::string band = gemm_epilogue(ki, sp, slot, "(QROW_ + mlc) * " + std::to_string(sp.LDC), {}, 0, rows,
                                           "(mlc / " + std::to_string(R) + ") * " + std::to_string(sp.WTM - R) + " + QOFF_", &inv);
    auto filled = [](std::string t, const std::string& from, int64_t v) {
      const std::string to = std::to_string(v);
      for (size_t i = t.find(from); i != std::string::npos; i = t.find(from, i + to.size())) t.replace(i, from.size(), to);
      return t;
    };
    s << inv;
    for (int q = 0; q < NQ; ++q) {
      s << "  {\n#pragma unroll\n  for (int i = 0; i < " << FQ << "; ++i)\n#pragma unroll\n  for (int j = 0; j < " << sp.FN
        << "; ++j)\n#pragma unroll\n  for (int r = 0; r < 4; ++r) Cs[(" << (q & 1) * rows << " + wm * " << R
        << " + i * 16 + (l >> 4) * 4 + r) * " << sp.LDC << " + wn * " << sp.WTN << " + j * 16 + (l & 15)] = acc[" << q * FQ
        << " + i][j][r];\n  }\n  __syncthreads();\n";
      s << filled(filled(band, "QROW_", (q & 1) * rows), "QOFF_", q * R);
    }
  }
  s << "  }\n}\n";
  gk.source = s.str();
  gk.grid[0] = (int)(tiles * sp.KS);
  gk.block[0] = sp.NT;
  gk.lds_bytes = (int)phased_smem(sp);
  ki.fill_cost(gk);
  return gk;
}

}  // namespace korch
