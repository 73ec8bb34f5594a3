// Output-stationary grouped GEMM on gfx950 MFMA.
//
// A launch is a list of output tiles.  Each tile owns a rectangle of one
// output matrix C and a contiguous range of segments; every segment adds
// alpha * A * B (A: m x k, B: k x n, either may be stored transposed) to the
// same tile, so all contributions to a tile accumulate in registers and the
// tile is written once.  No two tiles of one launch may overlap in C.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "common.h"

namespace dmrg {

enum SegFlags : int32_t {
  kTransA = 1,  // A stored k x m: A[i][k] = a[k * lda + i]
  kTransB = 2,  // B stored n x k: B[k][j] = b[j * ldb + k]
};

struct GemmSeg {
  const void* a;
  const void* b;
  int32_t lda, ldb, k, flags;
  double alpha;
};

struct GemmTile {
  void* c;
  int32_t ldc;
  int32_t m, n;        // valid rows / cols of this tile
  int32_t row0, col0;  // tile origin inside the problem (offsets A rows / B cols)
  int32_t seg_begin, seg_end;
  int32_t beta;        // 0: C = sum, 1: C += sum
  int32_t pad;         // k-split launches: the tile's first share
};

// Segments [s0, s1) of a tile's list, the share of one wave of the k-split
// kernel, and their 8-deep k-chunks in all.
struct GemmShare {
  int32_t s0, s1, chunks, pad;
};
constexpr int kKsTile = 64, kKsWaves = 4;  // output tile edge and waves of the k-split kernel

// A tile of one NT product (one segment), up to kOneRows x kOneCols, for the
// single-product kernel: operands and output at the tile's origin.
struct GemmOne {
  const void *a, *b;
  void* c;
  double alpha;
  int32_t lda, ldb, ldc, m, n, k;
  int32_t problem, pad;  // host side: the output problem
};
constexpr int kOneRows = 64, kOneCols = 256;
// its small form, for launches of at most 32 rows: a wave takes a whole tile,
// a workgroup the next kOneWaves of the list
constexpr int kOneSmall = 32, kOneWaves = 4;
inline int one_small_cols(int rows) { return rows <= 16 ? 64 : 32; }

constexpr int kTileM = 64;
constexpr int kTileN = 64;

// Host-side accumulation of one launch.
struct GemmBatch {
  std::vector<GemmSeg> segs;
  std::vector<GemmTile> tiles;
  double flops = 0;  // algorithmic 2*m*n*k over all segments
  // output tile of the launch (rows x cols): 64 x 64 (4 waves), 128 x 128,
  // 128 x 64 or 64 x 128 (8 waves)
  int tile = kTileM, tile_n = kTileN;
  // run on the k-split kernel (64 x 64 tiles, NT segments) where the operands
  // allow: each tile's `pad` names the first of its kKsWaves shares
  bool ksplit = false;
  bool raw = false;  // k-split: A rows as a caller stores them (any stride and alignment, ending at k)
  std::vector<GemmShare> shares;

  // Adds one output problem C (m x n, ldc) += sum over segs [s0, s1).
  // The problem is split into tile x tile_n pieces that share the segments.
  void add_problem(void* c, int ldc, int m, int n, size_t s0, size_t s1, int beta) {
    if (m <= 0 || n <= 0 || s1 <= s0) return;
    const int share = ksplit ? share_out(s0, s1) : 0;
    // k-split tiles cut an edge into nearly equal runs of whole 16-blocks:
    // their time follows the valid blocks
    const int tm = ksplit ? even_step(m, kKsTile) : tile, tn = ksplit ? even_step(n, kKsTile) : tile_n;
    for (int r = 0; r < m; r += tm)
      for (int q = 0; q < n; q += tn) {
        GemmTile t;
        t.c = c;
        t.ldc = ldc;
        t.m = std::min(tm, m - r);
        t.n = std::min(tn, n - q);
        t.row0 = r;
        t.col0 = q;
        t.seg_begin = (int32_t)s0;
        t.seg_end = (int32_t)s1;
        t.beta = beta;
        t.pad = share;
        tiles.push_back(t);
      }
    for (size_t s = s0; s < s1; ++s) flops += 2.0 * m * n * segs[s].k;
  }
  // Cuts segments [s0, s1) into kKsWaves shares of about equal k.
  int share_out(size_t s0, size_t s1) {
    constexpr int n = kKsWaves;
    int64_t total = 0, acc = 0;
    for (size_t s = s0; s < s1; ++s) total += (segs[s].k + 7) / 8;
    const int at = (int)shares.size();
    GemmShare w{(int32_t)s0, (int32_t)s0, 0, 0};
    for (int q = 0; q < n; ++q) {
      while (w.s1 < (int32_t)s1 && (q == n - 1 || acc * n < total * (q + 1))) {
        const int c = (segs[w.s1].k + 7) / 8;
        // a segment goes to the share that holds its middle
        if (q < n - 1 && (2 * acc + c) * n > 2 * total * (q + 1)) break;
        acc += c;
        w.chunks += c;
        ++w.s1;
      }
      shares.push_back(w);
      w = GemmShare{w.s1, w.s1, 0, 0};
    }
    return at;
  }
  static int even_step(int m, int tile) {
    const int parts = (m + tile - 1) / tile, blocks = (m + 15) / 16;
    return 16 * ((blocks + parts - 1) / parts);
  }
  void clear() { segs.clear(); tiles.clear(); shares.clear(); flops = 0; }
};

// MI355X hands the workgroups of a launch to its 8 XCDs round-robin by block
// index (block b runs on XCD b mod 8), and each XCD has its own L2.
constexpr int kXcds = 8;

// Reorders a launch's tiles for L2 locality.  key[t] names a locality group
// (tiles of one group share operands: the caller emits them consecutively,
// problem by problem, each problem's tiles row by row).  A group runs on one
// XCD, in emission order; groups are spread over the XCDs longest first onto
// the least loaded one, a group larger than a quarter of an XCD's share being
// cut at problem boundaries into pieces of about that size (cost(tile)
// estimates a tile's time).  Queues are interleaved so that block b takes the
// next tile of XCD b mod 8's queue; shorter queues are padded with empty
// tiles (m = 0), which the kernels skip.
// per: tiles that one workgroup takes.
template <class Tile, class Cost, class Same>
void xcd_order(std::vector<Tile>& tiles, const std::vector<int>& key, Cost&& cost, Same&& same, int per = 1) {
  struct Group {
    size_t t0, t1;
    double c;
  };
  const size_t nt = tiles.size();
  std::vector<double> tc(nt);
  double total = 0;
  for (size_t i = 0; i < nt; ++i) total += (tc[i] = cost(tiles[i]));
  const double cap = std::max(1.0, total / (4.0 * kXcds));
  auto same_problem = [&](size_t a, size_t b) { return same(tiles[a], tiles[b]); };
  std::vector<Group> groups;
  for (size_t i = 0; i < nt;) {
    size_t j = i;
    double c = 0;
    // extend over whole problems of the same key up to the cap
    while (j < nt && key[j] == key[i]) {
      size_t e = j + 1;
      while (e < nt && same_problem(e, j)) ++e;
      double pc = 0;
      for (size_t k = j; k < e; ++k) pc += tc[k];
      if (j > i && c + pc > cap) break;
      c += pc;
      j = e;
    }
    groups.push_back({i, j, c});
    i = j;
  }
  std::stable_sort(groups.begin(), groups.end(), [](const Group& a, const Group& b) { return a.c > b.c; });
  std::vector<std::vector<size_t>> queue(kXcds);
  double load[kXcds] = {};
  for (const Group& g : groups) {
    int x = 0;
    for (int y = 1; y < kXcds; ++y)
      if (load[y] < load[x]) x = y;
    for (size_t k = g.t0; k < g.t1; ++k) queue[x].push_back(k);
    load[x] += g.c;
  }
  size_t len = 0;
  for (auto& q : queue) len = std::max(len, q.size());
  Tile empty{};
  std::vector<Tile> out;
  out.reserve((len + per) * kXcds);
  for (size_t i = 0; i < len; i += per)
    for (int x = 0; x < kXcds; ++x)
      for (size_t j = i; j < i + per; ++j) out.push_back(j < queue[x].size() ? tiles[queue[x][j]] : empty);
  tiles.swap(out);
}
template <class Tile, class Cost>
void xcd_order(std::vector<Tile>& tiles, const std::vector<int>& key, Cost&& cost) {
  xcd_order(tiles, key, cost, [](const Tile& a, const Tile& b) {
    return a.c == b.c && a.seg_begin == b.seg_begin && a.seg_end == b.seg_end;
  });
}

// Launch (stream-ordered, no host synchronisation).  The descriptors are
// copied into pinned staging memory of the library, so the caller may
// release b as soon as the call returns; operand and output buffers must stay
// valid until the launch has run.
void launch_gemm_f64(const GemmBatch& b, hipStream_t stream);

// Descriptors uploaded once and launched many times (no host work per launch).
struct DevGemm {
  DevBuf buf;
  GemmSeg* segs = nullptr;
  GemmTile* tiles = nullptr;
  GemmShare* shares = nullptr;
  size_t ntiles = 0, nsegs = 0;
  double flops = 0;
  int tile = kTileM, tile_n = kTileN;
  bool lds = false;  // every segment suits the direct-to-LDS kernels
  bool ksplit = false, raw = false;
  bool small = false;  // k-split: tiles of at most 32 x 32; single products: at most 32 rows
  GemmOne* ones = nullptr;  // single-product launches (instead of tiles and segs)
};
void upload_gemm(const GemmBatch& b, DevGemm& d);
// Whether an NT product (16-byte aligned operands) suits the kernels that take
// fragments straight from global memory: rows readable up to a multiple of 8
// entries, a tile's rows within 32-bit byte offsets.
inline bool f64_direct_ok(int lda, int ldb, int k) {
  return lda % 8 == 0 && ldb % 8 == 0 && k > 0 && std::max(lda, ldb) < 1 << 20;
}
// raw: as GemmBatch::raw; small: tiles for the small form
void upload_gemm(const std::vector<GemmOne>& b, DevGemm& d, bool small, bool raw = false);
void launch_gemm_f64(const DevGemm& d, hipStream_t stream, int role = 0);

// ---- elementwise / BLAS-1 helpers (FP64) ----------------------------------
void launch_scale(double* x, double a, int64_t n, hipStream_t s);
void launch_axpy(double* y, double a, const double* x, int64_t n, hipStream_t s);
void launch_fill(double* x, double v, int64_t n, hipStream_t s);
// z = a x + b y (z may alias x or y)
void launch_axpby(double* z, double a, const double* x, double b, const double* y, int64_t n,
                  hipStream_t s);
// out[j] = sum_i X[j][i] * y[i] for j < nv (X rows of length n, row stride ldx)
void launch_multidot(double* out, const double* X, int64_t ldx, int nv, const double* y,
                     int64_t n, hipStream_t s);
// y = sum_j c[j] * X[j] (+ beta * y)
void launch_lincomb(double* y, const double* X, int64_t ldx, int nv, const double* c,
                    int64_t n, double beta, hipStream_t s, double alpha = 1.0);
// block copies (one workgroup per task), optionally transposing
struct CopyTask;
void launch_copy_tasks(const CopyTask* tasks, int ntasks, bool transpose, hipStream_t s);
// the sigma's way in and out of the padded layout (one workgroup per task)
struct PackTask;
struct PackMore;
struct SumTask;
void launch_pack_psi(const PackTask* tasks, int ntasks, const double* psi, hipStream_t s, const PackMore& more);
void launch_unpack_sigma(const SumTask* tasks, int ntasks, double* sigma, hipStream_t s);
// scatter-add rows: dst[idx[r]] += src[r]   (rows of length n)
void launch_row_scatter_add(double* dst, const double* src, const int64_t* dst_off, int nrows,
                            int64_t n, hipStream_t s);

}  // namespace dmrg
