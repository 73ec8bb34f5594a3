// gfx950 kernels: FP64-MFMA grouped GEMM and FP64 BLAS-1 helpers.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>

#include <algorithm>
#include <type_traits>

#include "gemm.h"
#include "gemm_bf16.h"
#include "davidson.h"
#include "engine.h"

namespace dmrg {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// One workgroup per TM x TN output tile: 64 x 64 with 4 waves (each a
// 32 x 32 quarter as 2 x 2 blocks of v_mfma_f64_16x16x4f64), 128 x 128 with
// 8 waves (each 64 x 32 as 4 x 2 blocks; twice the operand reuse per loaded
// byte), or 128 x 64 / 64 x 128 with 8 waves of 32 x 32 (4/3 of the reuse at
// the register count of the 64 x 64 tile).
// Operands are staged through LDS in k-slabs of 16 with bounds-checked
// (zero-filled) loads, so ragged m, n, k need no padding in memory.  alpha is
// folded into A.  The slabs of all segments of a tile form one sequence,
// double-buffered: the global loads of the next slab are issued into
// registers before the MFMAs of the current one, then stored into the other
// LDS buffer (one barrier per slab).
//
// MFMA operand layout (16x16x4 f64, wave64): lane l supplies A[l%16][l/16]
// and B[l/16][l%16]; accumulator element v of lane l holds D[4*v + l/16][l%16]
// (rows interleaved across the four 16-lane groups).
constexpr int kTK = 16;
constexpr int f64_waves(int TM, int TN) { return TM == 64 && TN == 64 ? 4 : 8; }
constexpr int f64_wave_rows(int TM, int TN) { return TM == 128 && TN == 64 ? 4 : 2; }

// ROLE only names the kernel for profilers: 0 = operator construction,
// 1 = sigma stage 1 (psi x right operator), 2 = sigma stage 2 (left operator x T).
template <int ROLE, int TM, int TN>
__global__ __launch_bounds__(64 * f64_waves(TM, TN)) void k_gemm_f64(const GemmTile* __restrict__ tiles,
                                                                     const GemmSeg* __restrict__ segs) {
  constexpr int WV = f64_waves(TM, TN), NT = 64 * WV;
  constexpr int WR = f64_wave_rows(TM, TN), WC = WV / WR;  // waves down the rows / across the columns
  constexpr int FM = TM / (16 * WR), FN = TN / (16 * WC);  // 16x16 blocks of a wave
  constexpr int kLoadsA = (TM * kTK) / NT, kLoadsB = (TN * kTK) / NT;
  static_assert(FM >= 1 && FN >= 1 && kLoadsA >= 1 && kLoadsB >= 1, "k_gemm_f64: tile shape");
  __shared__ double As[2][kTK][TM + 1];
  __shared__ double Bs[2][kTK][TN + 1];
  const GemmTile t = tiles[blockIdx.x];
  if (t.m <= 0) return;  // padding tile of the XCD-ordered launch
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = (wave / WC) * (TM / WR), wn = (wave % WC) * (TN / WC);
  const int lr = lane & 15, lk = lane >> 4;
  f64x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};

  if (t.seg_begin < t.seg_end) {
    double ra[kLoadsA], rb[kLoadsB];
    // global loads of the slab at k offset k0 of segment g into ra, rb
    auto load = [&](const GemmSeg& g, int k0) {
      const double* __restrict__ A = static_cast<const double*>(g.a);
      const double* __restrict__ B = static_cast<const double*>(g.b);
      const bool ta = g.flags & kTransA, tb = g.flags & kTransB;
#pragma unroll
      for (int r = 0; r < kLoadsA; ++r) {
        const int e = r * NT + tid;
        int i, kk;
        if (!ta) { i = e / kTK; kk = e % kTK; }
        else { kk = e / TM; i = e % TM; }
        const int gk = k0 + kk;
        double v = 0.0;
        if (i < t.m && gk < g.k) {
          const int64_t gi = (int64_t)t.row0 + i;
          v = ta ? A[(int64_t)gk * g.lda + gi] : A[gi * g.lda + gk];
        }
        ra[r] = v * g.alpha;
      }
#pragma unroll
      for (int r = 0; r < kLoadsB; ++r) {
        const int e = r * NT + tid;
        int j, kk;
        if (!tb) { kk = e / TN; j = e % TN; }
        else { j = e / kTK; kk = e % kTK; }
        const int gk = k0 + kk;
        double v = 0.0;
        if (j < t.n && gk < g.k) {
          const int64_t gj = (int64_t)t.col0 + j;
          v = tb ? B[gj * g.ldb + gk] : B[(int64_t)gk * g.ldb + gj];
        }
        rb[r] = v;
      }
    };
    // ra, rb into LDS buffer buf (same element placement as the loads)
    auto store = [&](const GemmSeg& g, int buf) {
      const bool ta = g.flags & kTransA, tb = g.flags & kTransB;
#pragma unroll
      for (int r = 0; r < kLoadsA; ++r) {
        const int e = r * NT + tid;
        if (!ta) As[buf][e % kTK][e / kTK] = ra[r];
        else As[buf][e / TM][e % TM] = ra[r];
      }
#pragma unroll
      for (int r = 0; r < kLoadsB; ++r) {
        const int e = r * NT + tid;
        if (!tb) Bs[buf][e / TN][e % TN] = rb[r];
        else Bs[buf][e % kTK][e / kTK] = rb[r];
      }
    };
    int s = t.seg_begin, k0 = 0, buf = 0;
    GemmSeg g = segs[s];
    load(g, 0);
    store(g, 0);
    __syncthreads();
    while (true) {
      // position of the next slab in the tile's sequence
      int ns = s, nk0 = k0 + kTK;
      GemmSeg ng = g;
      if (nk0 >= g.k) {
        nk0 = 0;
        if (++ns < t.seg_end) ng = segs[ns];
      }
      const bool more = ns < t.seg_end;
      if (more) load(ng, nk0);  // in flight during the MFMAs below
      // MFMAs only on 16x16 blocks and k-steps of 4 that meet the tile's
      // valid rows, columns and the segment's k (the rest of the LDS slab is
      // zero padding); the conditions are uniform over the wave, so the
      // skipped MFMAs leave the SIMD's matrix pipe to the other waves
      if (wm < t.m && wn < t.n) {
        const int kv = g.k - k0;  // valid k of this slab (>= 1)
#pragma unroll
        for (int kk = 0; kk < kTK; kk += 4) {
          if (kk >= kv) break;
          double a[FM], b[FN];
#pragma unroll
          for (int i = 0; i < FM; ++i) a[i] = As[buf][kk + lk][wm + 16 * i + lr];
#pragma unroll
          for (int j = 0; j < FN; ++j) b[j] = Bs[buf][kk + lk][wn + 16 * j + lr];
#pragma unroll
          for (int i = 0; i < FM; ++i)
            if (wm + 16 * i < t.m)
#pragma unroll
              for (int j = 0; j < FN; ++j)
                if (wn + 16 * j < t.n)
                  acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
      }
      if (!more) break;
      // the other buffer was last read before the previous barrier
      store(ng, buf ^ 1);
      __syncthreads();
      buf ^= 1;
      s = ns;
      k0 = nk0;
      g = ng;
    }
  }
  double* __restrict__ C = static_cast<double*>(t.c);
#pragma unroll
  for (int bi = 0; bi < FM; ++bi)
#pragma unroll
    for (int bj = 0; bj < FN; ++bj)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = wm + bi * 16 + 4 * v + lk;
        const int j = wn + bj * 16 + lr;
        if (i < t.m && j < t.n) {
          double* p = C + ((int64_t)t.row0 + i) * t.ldc + (t.col0 + j);
          const double val = acc[bi][bj][v];
          *p = t.beta ? (*p + val) : val;
        }
      }
}

// Direct-to-LDS variant for NT segments (A m x k and B stored n x k, both k
// contiguous, with even leading dimensions and 16-byte aligned bases, so
// that every 16-byte chunk of a row lies inside the row).  Each lane moves 16
// bytes of a slab from global memory straight into LDS (global_load_lds): no
// registers stage the operands, and a ring of three LDS stages keeps two
// slabs in flight during the MFMAs of a third (two stages for 128 x 128, so
// that two workgroups fit a CU).  A slab holds kTK = 16 k of
// the TM rows of A and the TN rows of B, 128 bytes a row; chunk c (k 2c,
// 2c + 1) of LDS row r sits at position c ^ ((r >> 1) & 7), so that the
// fragment reads of 16 consecutive rows at one k (half a wave) meet each
// bank once.  Chunks outside the operands read a zero buffer; k entries past
// a segment's k that share a chunk with valid ones are zeroed in the
// fragments, and alpha scales the A fragments.  The MFMA sequence (k-steps of
// 4, segment by segment) is that of k_gemm_f64, so both give the same bits.
__device__ __attribute__((aligned(16))) double g_f64_zero[2];  // 16 zero bytes (static storage)

template <int N>
__device__ __forceinline__ void f64_wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  // gfx9 encoding of s_waitcnt: vmcnt low bits [3:0], high bits [15:14];
  // expcnt and lgkmcnt at their maxima (not waited on)
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ int f64_swz(int row) { return (row >> 1) & 7; }

template <int ROLE, int TM, int TN>
__global__ __launch_bounds__(64 * f64_waves(TM, TN)) void k_gemm_f64_lds(const GemmTile* __restrict__ tiles,
                                                                         const GemmSeg* __restrict__ segs) {
  constexpr int WV = f64_waves(TM, TN);
  constexpr int WR = f64_wave_rows(TM, TN), WC = WV / WR;
  constexpr int FM = TM / (16 * WR), FN = TN / (16 * WC);
  constexpr int ROWS = TM + TN;        // 128-byte LDS rows of a slab
  constexpr int NL = ROWS / (8 * WV);  // wave loads (8 rows each) per wave and slab
  static_assert(NL >= 1 && NL * 8 * WV == ROWS && kTK == 16, "k_gemm_f64_lds: slab layout");
  // three LDS stages where two workgroups still fit a CU, else two
  constexpr int ST = 3 * ROWS * kTK * 8 <= 80 * 1024 ? 3 : 2;
  __shared__ __attribute__((aligned(16))) double sm[ST][ROWS * kTK];
  const GemmTile t = tiles[blockIdx.x];
  if (t.m <= 0) return;  // padding tile of the XCD-ordered launch
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = (wave / WC) * (TM / WR), wn = (wave % WC) * (TN / WC);
  const int lr = lane & 15, lk = lane >> 4;
  f64x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};

  if (t.seg_begin < t.seg_end) {
    // load j of a lane: LDS row 8 (wave NL + j) + lane / 8, position lane % 8
    const double* src[NL];
    int kc[NL];
    auto segment = [&](const GemmSeg& g) {
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const int r = 8 * (wave * NL + j) + (lane >> 3);
        const int c = (lane & 7) ^ f64_swz(r);
        kc[j] = 2 * c;
        if (r < TM)
          src[j] = r < t.m ? static_cast<const double*>(g.a) + (int64_t)(t.row0 + r) * g.lda + 2 * c : nullptr;
        else
          src[j] = r - TM < t.n ? static_cast<const double*>(g.b) + (int64_t)(t.col0 + r - TM) * g.ldb + 2 * c
                                : nullptr;
      }
    };
    int ps = t.seg_begin, pk0 = 0;
    GemmSeg pg = segs[ps];
    segment(pg);
    int cs = ps, ck0 = 0;
    GemmSeg cg = pg;
    int issued = 0, done = 0;
    auto produce = [&]() {
      double* buf = &sm[issued % ST][0];
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const double* p = (src[j] && pk0 + kc[j] < pg.k) ? src[j] + pk0 : g_f64_zero;
        __builtin_amdgcn_global_load_lds(p, buf + 128 * (wave * NL + j), 16, 0, 0);
      }
      ++issued;
      pk0 += kTK;
      if (pk0 >= pg.k) {
        pk0 = 0;
        if (++ps < t.seg_end) {
          pg = segs[ps];
          segment(pg);
        }
      }
    };
    produce();
    if (ST == 3 && ps < t.seg_end) produce();
    while (cs < t.seg_end) {
      // slab `done` is complete once at most ST - 2 newer slabs are pending
      if (ST == 3 && issued > done + 1) f64_wait_vm<NL>();
      else f64_wait_vm<0>();
      // barrier without a memory fence: every wave's loads of this slab are
      // in LDS, and every wave has read the buffer the next load overwrites
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (ps < t.seg_end) produce();
      const double* st = &sm[done % ST][0];
      if (wm < t.m && wn < t.n) {
        const int kv = cg.k - ck0;  // valid k of this slab
#pragma unroll
        for (int kk = 0; kk < kTK; kk += 4) {
          if (kk >= kv) break;
          const int k = kk + lk, c = k >> 1, h = k & 1;
          double a[FM], b[FN];
#pragma unroll
          for (int i = 0; i < FM; ++i) {
            const int r = wm + 16 * i + lr;
            a[i] = st[r * kTK + 2 * (c ^ f64_swz(r)) + h];
          }
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const int r = TM + wn + 16 * j + lr;
            b[j] = st[r * kTK + 2 * (c ^ f64_swz(r)) + h];
          }
          if (kv - kk < 4) {  // the segment's last k-step: entries past k are zero
            const bool ok = k < kv;
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = ok ? a[i] : 0.0;
#pragma unroll
            for (int j = 0; j < FN; ++j) b[j] = ok ? b[j] : 0.0;
          }
#pragma unroll
          for (int i = 0; i < FM; ++i) a[i] *= cg.alpha;
#pragma unroll
          for (int i = 0; i < FM; ++i)
            if (wm + 16 * i < t.m)
#pragma unroll
              for (int j = 0; j < FN; ++j)
                if (wn + 16 * j < t.n)
                  acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
      }
      ++done;
      ck0 += kTK;
      if (ck0 >= cg.k) {
        ck0 = 0;
        if (++cs < t.seg_end) cg = segs[cs];
      }
    }
  }
  double* __restrict__ C = static_cast<double*>(t.c);
#pragma unroll
  for (int bi = 0; bi < FM; ++bi)
#pragma unroll
    for (int bj = 0; bj < FN; ++bj)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = wm + bi * 16 + 4 * v + lk;
        const int j = wn + bj * 16 + lr;
        if (i < t.m && j < t.n) {
          double* p = C + ((int64_t)t.row0 + i) * t.ldc + (t.col0 + j);
          const double val = acc[bi][bj][v];
          *p = t.beta ? (*p + val) : val;
        }
      }
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) char* global_bytes;
typedef const __attribute__((address_space(1))) f64x2* global_f64x2;
typedef f64x2 f64x2_at8 __attribute__((aligned(8)));
typedef const __attribute__((address_space(1))) f64x2_at8* global_f64x2_at8;

// A lane's two entries (k = 2 lk, 2 lk + 1) of a row's 8-deep chunk, `valid`
// of them in the row.  RAW: rows of any stride and 8-byte alignment that end
// at their k >= 2; lanes past the end load the last two entries (of the row,
// so the address may lie before the chunk).  Else 16-byte aligned rows that
// are readable up to a multiple of 8.
template <bool RAW>
__device__ __forceinline__ f64x2 f64_pair(global_bytes p, uint32_t row, int lk, int valid) {
  if constexpr (RAW) return *(global_f64x2_at8)((p - 16) + (row + (uint32_t)(16 + 8 * min(2 * lk, valid - 2))));
  else return *(global_f64x2)(p + row);
}
// Entry q of the pair in a chunk with kv < 8 valid entries (before those past
// the end are zeroed): at an odd end the last entry is the pair's second.
template <bool RAW>
__device__ __forceinline__ double f64_tail(f64x2 x, int q, int lk, int kv) {
  return RAW && q == 0 && 2 * lk == kv - 1 ? x[1] : x[q];
}

// Share of one wave in a tile of FM x FN blocks of 16 x 16 (k_gemm_f64_ks):
// segments [sh.s0, sh.s1), sh.chunks chunks of 8 k in all.  A lane loads two
// consecutive entries of each of its fragment rows (the four lanes of a row
// take 64 consecutive bytes), which feed two MFMA k-steps; the loads of the
// next NST - 1 chunks are in flight, in registers, during a chunk's MFMAs.
// Every chunk issues its loads unconditionally (past the end they repeat the
// last segment), so that the waits before a chunk's MFMAs count only its own.
template <int FM, int FN, int NST, bool RAW>
__device__ __forceinline__ void f64_ks_share(const GemmTile& t, const GemmSeg* __restrict__ segs, const GemmShare sh,
                                             f64x4 (&acc)[FM][FN]) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  uint32_t ra[FM], rb[FN];  // fragment rows, kept inside the tile
#pragma unroll
  for (int i = 0; i < FM; ++i) ra[i] = (uint32_t)min(16 * i + lr, t.m - 1);
#pragma unroll
  for (int j = 0; j < FN; ++j) rb[j] = (uint32_t)min(16 * j + lr, t.n - 1);
  uint32_t oa[FM], ob[FN];  // byte offsets of a lane's loads from the operands' current k
  global_bytes pa, pb;
  int ps = sh.s0, left;
  double scale;
  auto segment = [&](const GemmSeg& g) {
    pa = (global_bytes)g.a + 8 * (int64_t)t.row0 * g.lda;
    pb = (global_bytes)g.b + 8 * (int64_t)t.col0 * g.ldb;
    left = g.k;
    scale = g.alpha;
#pragma unroll
    for (int i = 0; i < FM; ++i) oa[i] = 8 * ra[i] * (uint32_t)g.lda + (RAW ? 0 : 16 * lk);
#pragma unroll
    for (int j = 0; j < FN; ++j) ob[j] = 8 * rb[j] * (uint32_t)g.ldb + 16 * lk;
  };
  segment(segs[ps]);
  GemmSeg next = segs[min(ps + 1, sh.s1 - 1)];
  f64x2 fa[NST][FM], fb[NST][FN];
  double al[NST];
  int kv[NST];  // valid k of the chunk
  auto load = [&](int s) {
    al[s] = scale;
    kv[s] = left;
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[s][i] = f64_pair<RAW>(pa, oa[i], lk, left);
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[s][j] = *(global_f64x2)(pb + ob[j]);
    pa += 64;
    pb += 64;
    left -= 8;
    if (left <= 0) {
      ++ps;
      segment(next);
      next = segs[min(ps + 1, sh.s1 - 1)];
    }
  };
#pragma unroll
  for (int s = 0; s < NST; ++s) load(s);
  // whole rounds of NST chunks (one exit, so that the accumulators keep their
  // registers); those past the end are only loaded
  int todo = sh.chunks;
  do {
#pragma unroll
    for (int s = 0; s < NST; ++s) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (s >= todo) break;
        double a[FM], b[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) a[i] = fa[s][i][q] * al[s];
#pragma unroll
        for (int j = 0; j < FN; ++j) b[j] = fb[s][j][q];
        if (kv[s] < 8) {  // the segment's last chunk: entries past k are zero
          const bool ok = 2 * lk + q < kv[s];
#pragma unroll
          for (int i = 0; i < FM; ++i) a[i] = ok ? f64_tail<RAW>(fa[s][i], q, lk, kv[s]) * al[s] : 0.0;
#pragma unroll
          for (int j = 0; j < FN; ++j) b[j] = ok ? b[j] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      load(s);
    }
    todo -= NST;
  } while (todo > 0);
}

// Variant for long segment lists (sigma stage 2): the four waves of a
// workgroup each cover the whole tile (at most 64 x 64) and share out its
// segments.  An FP64 16x16x4 MFMA takes 64 cycles and no other VALU
// instruction of its SIMD runs beside it (measured: the times add up, also
// across waves), so the kernel spends as few instructions per MFMA as it can:
// no LDS, no barrier, fragments straight from the L1 in the MFMA layout, one
// pointer step per operand and chunk, and code for the tile's exact number
// of 16-blocks (f64_ks_share).  All waves issue equal MFMA counts whatever
// the tile's valid rows and columns are.  Operand rows must be readable up to
// a multiple of 8 entries.  At the end the four partial tiles are added
// through LDS, block row by block row, in wave order.
//
// Stage 2 of one sigma, before (k_gemm_f64_lds, a workgroup per 128 x 64
// tile and whole list) and now, ms: 8 orbitals D = 64 0.25 -> 0.022; 16
// orbitals D = 512 2.60 -> 0.52; 22 orbitals D = 1024 16.9 -> 4.3; 15
// orbitals D = 3001 46.0 -> 30.  Most of that is the split of the lists over
// the chip; of the kernel's forms, the same split with slabs in LDS and a
// barrier each took 0.67 ms at 16 orbitals and 6.8 ms at 22.  What bounds it
// now is the traffic beyond the L2 (28 GB at 22 orbitals, 5.4 TB/s; without
// it the launch takes 3.7 ms), MFMA pipes 63% busy there and 81% at the
// smallest chunks of 15 orbitals.
// SMALL: every tile of the launch has at most 32 rows and columns (four
// workgroups a CU instead of two).
// RAW: A rows as the caller stores them (f64_pair; spin-adapted sigma, 6 + 6
// orbitals' pairs on 2048 multiplets a side: k_gemm_f64 1.87 ms, now 1.17;
// 1.26 with two 8-byte loads a pair, 1.08 with padded copies of the blocks,
// which would double the operators' memory).
template <int ROLE, bool SMALL, bool RAW>
__global__ __launch_bounds__(64 * kKsWaves, SMALL ? 4 : 2) void k_gemm_f64_ks(const GemmTile* __restrict__ tiles,
                                                                  const GemmSeg* __restrict__ segs,
                                                                  const GemmShare* __restrict__ shares) {
  constexpr int RS = (SMALL ? 32 : kKsTile) + 16;  // row stride of the partial sums in LDS
  __shared__ double sm[kKsWaves * 16 * RS];
  const GemmTile t = tiles[blockIdx.x];
  if (t.m <= 0) return;  // padding tile of the XCD-ordered launch
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lr = lane & 15, lk = lane >> 4;
  const int bm = (t.m + 15) >> 4, bn = (t.n + 15) >> 4;
  const GemmShare sh = shares[t.pad + wave];
  double* __restrict__ C = static_cast<double*>(t.c);
  auto store = [&](int r, int c, double val) {
    if (r < t.m && c < t.n) {
      double* p = C + ((int64_t)t.row0 + r) * t.ldc + (t.col0 + c);
      *p = t.beta ? *p + val : val;
    }
  };
  // block row i of the four partial tiles in LDS: their sum
  auto finish = [&](int i) {
    __syncthreads();
    for (int c = tid & 15; c < t.n; c += 16) {
      const double* q = sm + (tid >> 4) * RS + c;
      double val = q[0];
#pragma unroll
      for (int w = 1; w < kKsWaves; ++w) val += q[w * 16 * RS];
      store(16 * i + (tid >> 4), c, val);
    }
    __syncthreads();
  };
#define DMRG_KS(FM, FN, NST)                                                                        \
  case FM * 8 + FN: {                                                                               \
    f64x4 acc[FM][FN];                                                                              \
    _Pragma("unroll") for (int i = 0; i < FM; ++i)                                                  \
      _Pragma("unroll") for (int j = 0; j < FN; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};         \
    if (sh.chunks > 0) f64_ks_share<FM, FN, NST, RAW>(t, segs, sh, acc);                                 \
    _Pragma("unroll") for (int i = 0; i < FM; ++i) {                                                \
      _Pragma("unroll") for (int j = 0; j < FN; ++j)                                                \
        _Pragma("unroll") for (int v = 0; v < 4; ++v)                                               \
          sm[(wave * 16 + 4 * v + lk) * RS + 16 * j + lr] = acc[i][j][v];                           \
      finish(i);                                                                                    \
    }                                                                                               \
    break;                                                                                          \
  }
  static_assert(kKsTile == 64, "k_gemm_f64_ks: the shapes below cover 64 x 64");
  if constexpr (SMALL) {
    switch (bm * 8 + bn) { DMRG_KS(2, 2, 3) DMRG_KS(2, 1, 4) DMRG_KS(1, 2, 4) DMRG_KS(1, 1, 6) }
  } else {
  switch (bm * 8 + bn) {
    DMRG_KS(4, 4, 2) DMRG_KS(4, 3, 2) DMRG_KS(4, 2, 3) DMRG_KS(4, 1, 4)
    DMRG_KS(3, 4, 2) DMRG_KS(3, 3, 3) DMRG_KS(3, 2, 3) DMRG_KS(3, 1, 4)
    DMRG_KS(2, 4, 3) DMRG_KS(2, 3, 3) DMRG_KS(2, 2, 4) DMRG_KS(2, 1, 6)
    DMRG_KS(1, 4, 4) DMRG_KS(1, 3, 4) DMRG_KS(1, 2, 6) DMRG_KS(1, 1, 8)
  }
  }
#undef DMRG_KS
}

// Single products (sigma stage 1): a tile of at most 64 x 256 of one NT
// product, its columns dealt to four waves in whole 16-blocks.  As in
// k_gemm_f64_ks the fragments come straight from the L1 in the MFMA layout
// (the waves share the A rows), the next chunks' loads in flight during a
// chunk's MFMAs, with code for each wave's exact number of 16-blocks; one
// descriptor holds all a tile needs, so a wave's first loads wait for one
// read.  Stage 1 of one sigma, before (k_gemm_f64_lds, 128 x 128) and now,
// ms: 8 orbitals D = 64 0.023 -> 0.017; 16 orbitals D = 512 0.50 -> 0.43; 22
// orbitals D = 1024 3.4 -> 3.3 (5.5 GB written; 2.6 without the stores, 2.7
// without the loads, 3.1 without the MFMAs: no one of them bounds it); 15
// orbitals D = 3001 18.2 -> 15.5 (49 TFLOP/s).  Sweeping a wave over more
// columns as one stream of chunks was slower (15 orbitals 18.8 ms).
template <int FM, int FN, int NST, bool RAW>
__device__ __forceinline__ void f64_one_tile(const GemmOne& t, int c0, int nc) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  uint32_t oa[FM], ob[FN];  // byte offsets of a lane's loads from the operands' current k
#pragma unroll
  for (int i = 0; i < FM; ++i) oa[i] = 8 * (uint32_t)min(16 * i + lr, t.m - 1) * (uint32_t)t.lda + (RAW ? 0 : 16 * lk);
#pragma unroll
  for (int j = 0; j < FN; ++j) ob[j] = 8 * (uint32_t)min(16 * j + lr, nc - 1) * (uint32_t)t.ldb + 16 * lk;
  global_bytes pa = (global_bytes)t.a, pb = (global_bytes)t.b + 8 * (int64_t)c0 * t.ldb;
  f64x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  f64x2 fa[NST][FM], fb[NST][FN];
  int left = t.k;  // k from the chunk to load on; the last one is loaded again past the end
  auto load = [&](int s) {
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[s][i] = f64_pair<RAW>(pa, oa[i], lk, left);
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[s][j] = *(global_f64x2)(pb + ob[j]);
    const int step = left > 8 ? 8 : 0;
    pa += 8 * step;
    pb += 8 * step;
    left -= step;
  };
#pragma unroll
  for (int s = 0; s < NST; ++s) load(s);
  int k = t.k;  // k not multiplied yet
  do {
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      const int kv = k - 8 * s;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (kv <= 0) break;
        double a[FM], b[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) a[i] = fa[s][i][q];
#pragma unroll
        for (int j = 0; j < FN; ++j) b[j] = fb[s][j][q];
        if (kv < 8) {  // the last chunk: entries past k are zero
          const bool ok = 2 * lk + q < kv;
#pragma unroll
          for (int i = 0; i < FM; ++i) a[i] = ok ? f64_tail<RAW>(fa[s][i], q, lk, kv) : 0.0;
#pragma unroll
          for (int j = 0; j < FN; ++j) b[j] = ok ? b[j] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      load(s);
    }
    k -= 8 * NST;
  } while (k > 0);
  double* __restrict__ C = static_cast<double*>(t.c) + c0;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * i + 4 * v + lk;
      if (r >= t.m) continue;
      double* row = C + (int64_t)r * t.ldc;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int c = 16 * j + lr;
        if (c >= nc) continue;
        row[c] = t.alpha * acc[i][j][v];
      }
    }
}

// SMALL: tiles of at most 32 x 32 or 16 x 64, one a wave (four workgroups a CU instead of
// two): small blocks leave too few columns for four waves, and a tile is a
// chain of latencies (8 orbitals D = 64: 21 us with the columns of a tile
// dealt to the waves of a workgroup, 19.5 with 32 x 32 only, now 17; 12
// orbitals D = 256 121 -> 96).  RAW: A rows as the caller stores them (f64_pair; spin-adapted stage 1 as above, 1.1 GB written:
// k_gemm_f64 0.85 ms, now 0.68).
template <int ROLE, bool SMALL, bool RAW>
__global__ __launch_bounds__(64 * kOneWaves, SMALL ? 4 : 2) void k_gemm_f64_one(const GemmOne* __restrict__ tiles) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const GemmOne t = tiles[SMALL ? kOneWaves * blockIdx.x + wave : blockIdx.x];
  if (t.m <= 0) return;  // padding tile of the XCD-ordered launch
  const int nb = (t.n + 15) >> 4, b0 = SMALL ? 0 : (nb * wave) >> 2, b1 = SMALL ? nb : (nb * (wave + 1)) >> 2;
  if (b0 == b1) return;
  const int c0 = 16 * b0, nc = min(t.n, 16 * b1) - c0;
#define DMRG_ONE(FM, FN, NST) \
  case FM * 8 + FN:           \
    f64_one_tile<FM, FN, NST, RAW>(t, c0, nc); \
    break;
  static_assert(kOneRows == 64 && kOneCols == 256 && kOneSmall == 32 && kOneWaves == 4,
                "k_gemm_f64_one: the shapes below cover 64 x 64 a wave, SMALL 32 x 32");
  const int shape = ((t.m + 15) >> 4) * 8 + b1 - b0;
  if constexpr (SMALL) {
    switch (shape) {
      DMRG_ONE(2, 2, 3) DMRG_ONE(2, 1, 4)
      DMRG_ONE(1, 4, 3) DMRG_ONE(1, 3, 3) DMRG_ONE(1, 2, 4) DMRG_ONE(1, 1, 4)
    }
    return;
  }
  switch (shape) {
    DMRG_ONE(4, 4, 2) DMRG_ONE(4, 3, 2) DMRG_ONE(4, 2, 2) DMRG_ONE(4, 1, 3)
    DMRG_ONE(3, 4, 2) DMRG_ONE(3, 3, 2) DMRG_ONE(3, 2, 3) DMRG_ONE(3, 1, 3)
    DMRG_ONE(2, 4, 2) DMRG_ONE(2, 3, 3) DMRG_ONE(2, 2, 3) DMRG_ONE(2, 1, 4)
    DMRG_ONE(1, 4, 3) DMRG_ONE(1, 3, 3) DMRG_ONE(1, 2, 4) DMRG_ONE(1, 1, 4)
  }
#undef DMRG_ONE
}

// Whether every segment of a launch suits k_gemm_f64_lds: NT operands with
// even leading dimensions and 16-byte aligned bases.  DMRG_F64_LDS=0 keeps
// every launch on k_gemm_f64.
static bool f64_lds_ok(const GemmSeg* segs, size_t n) {
  const char* e = std::getenv("DMRG_F64_LDS");
  if (e && std::atoi(e) == 0) return false;
  for (size_t i = 0; i < n; ++i) {
    const GemmSeg& g = segs[i];
    if ((g.flags & kTransA) || !(g.flags & kTransB) || (g.lda & 1) || (g.ldb & 1) ||
        (reinterpret_cast<uintptr_t>(g.a) & 15) || (reinterpret_cast<uintptr_t>(g.b) & 15))
      return false;
  }
  return true;
}

// One launch of cnt tiles of the given shape (rows x cols) and role.
static void launch_f64_tiles(int role, int tm, int tn, bool lds, unsigned cnt, hipStream_t s, const GemmTile* tiles,
                             const GemmSeg* segs) {
#define DMRG_LF(R, TM, TN)                                                                                       \
  do {                                                                                                          \
    if (lds)                                                                                                    \
      hipLaunchKernelGGL((k_gemm_f64_lds<R, TM, TN>), dim3(cnt), dim3(64 * f64_waves(TM, TN)), 0, s, tiles, segs); \
    else                                                                                                        \
      hipLaunchKernelGGL((k_gemm_f64<R, TM, TN>), dim3(cnt), dim3(64 * f64_waves(TM, TN)), 0, s, tiles, segs);     \
  } while (0)
#define DMRG_LF_ROLES(TM, TN)               \
  do {                                      \
    if (role == 1) DMRG_LF(1, TM, TN);      \
    else if (role == 2) DMRG_LF(2, TM, TN); \
    else DMRG_LF(0, TM, TN);                \
  } while (0)
  if (tm == 128 && tn == 128) DMRG_LF_ROLES(128, 128);
  else if (tm == 128 && tn == 64) DMRG_LF_ROLES(128, 64);
  else if (tm == 64 && tn == 128) DMRG_LF_ROLES(64, 128);
  else {
    DMRG_REQUIRE(tm == 64 && tn == 64, kErrInvalidArg, "k_gemm_f64: tile must be 64x64, 128x128, 128x64 or 64x128");
    DMRG_LF_ROLES(64, 64);
  }
#undef DMRG_LF_ROLES
#undef DMRG_LF
}

// Descriptors of one-off launches go through a ring of pinned host buffers
// copied asynchronously to device buffers, so that a launch needs no host
// synchronisation: a slot is reused only after the event recorded behind
// the launch that read it has completed.  One ring per device and host
// thread, kept until the process ends.
namespace {
struct DescSlot {
  char* host = nullptr;
  DevBuf dev;
  size_t cap = 0;
  hipEvent_t ev = nullptr;
  bool used = false;
};
constexpr int kDescSlots = 8;
struct DescRing {
  DescSlot slot[kDescSlots];
  int next = 0;
};
DescRing& desc_ring() {
  static thread_local std::map<int, DescRing*> rings;
  int dev = 0;
  DMRG_HIP(hipGetDevice(&dev));
  DescRing*& r = rings[dev];
  if (!r) r = new DescRing();  // process lifetime
  return *r;
}
}  // namespace

void launch_gemm_f64(const GemmBatch& b, hipStream_t stream) {
  if (b.tiles.empty()) return;
  const size_t sb = b.segs.size() * sizeof(GemmSeg);
  const size_t sba = ((sb + 255) / 256) * 256;
  const size_t tb = b.tiles.size() * sizeof(GemmTile);
  const size_t need = sba + tb;
  DescRing& ring = desc_ring();
  DescSlot& sl = ring.slot[ring.next];
  ring.next = (ring.next + 1) % kDescSlots;
  if (sl.used) DMRG_HIP(hipEventSynchronize(sl.ev));
  if (!sl.ev) DMRG_HIP(hipEventCreateWithFlags(&sl.ev, hipEventDisableTiming));
  if (sl.cap < need) {
    const size_t cap = std::max(need, (size_t)1 << 16);
    if (sl.host) DMRG_HIP(hipHostFree(sl.host));
    sl.host = nullptr;
    DMRG_HIP(hipHostMalloc(reinterpret_cast<void**>(&sl.host), cap));
    sl.dev.alloc(cap);
    sl.cap = cap;
  }
  std::memcpy(sl.host, b.segs.data(), sb);
  std::memcpy(sl.host + sba, b.tiles.data(), tb);
  DMRG_HIP(hipMemcpyAsync(sl.dev.p, sl.host, need, hipMemcpyHostToDevice, stream));
  GemmSeg* dsegs = sl.dev.as<GemmSeg>();
  GemmTile* dtiles = reinterpret_cast<GemmTile*>(sl.dev.as<char>() + sba);
  const size_t nt = b.tiles.size();
  const bool lds = f64_lds_ok(b.segs.data(), b.segs.size());
  for (size_t off = 0; off < nt; off += (size_t)1 << 30) {
    const unsigned cnt = (unsigned)std::min<size_t>(nt - off, (size_t)1 << 30);
    launch_f64_tiles(0, b.tile, b.tile_n, lds, cnt, stream, dtiles + off, dsegs);
  }
  DMRG_HIP(hipGetLastError());
  DMRG_HIP(hipEventRecord(sl.ev, stream));
  sl.used = true;
}

void upload_gemm(const GemmBatch& b, DevGemm& d) {
  const size_t sb = b.segs.size() * sizeof(GemmSeg);
  const size_t tb = b.tiles.size() * sizeof(GemmTile);
  const size_t sba = ((sb + 255) / 256) * 256;
  const size_t tba = ((tb + 255) / 256) * 256, hb = b.shares.size() * sizeof(GemmShare);
  d.buf.alloc(sba + tba + hb + 256);
  d.segs = reinterpret_cast<GemmSeg*>(d.buf.as<char>());
  d.tiles = reinterpret_cast<GemmTile*>(d.buf.as<char>() + sba);
  d.shares = reinterpret_cast<GemmShare*>(d.buf.as<char>() + sba + tba);
  if (hb) DMRG_HIP(hipMemcpy(d.shares, b.shares.data(), hb, hipMemcpyHostToDevice));
  if (sb) DMRG_HIP(hipMemcpy(d.segs, b.segs.data(), sb, hipMemcpyHostToDevice));
  if (tb) DMRG_HIP(hipMemcpy(d.tiles, b.tiles.data(), tb, hipMemcpyHostToDevice));
  d.ntiles = b.tiles.size();
  d.nsegs = b.segs.size();
  d.flops = b.flops;
  d.tile = b.tile;
  d.tile_n = b.tile_n;
  d.lds = f64_lds_ok(b.segs.data(), b.segs.size());
  d.ksplit = b.ksplit;
  d.raw = b.raw;
  d.small = true;
  for (const GemmTile& t : b.tiles) d.small = d.small && t.m <= 32 && t.n <= 32;
}

void upload_gemm(const std::vector<GemmOne>& b, DevGemm& d, bool small, bool raw) {
  d.raw = raw;
  d.buf.alloc(std::max<size_t>(1, b.size()) * sizeof(GemmOne));
  d.ones = d.buf.as<GemmOne>();
  if (!b.empty()) DMRG_HIP(hipMemcpy(d.ones, b.data(), b.size() * sizeof(GemmOne), hipMemcpyHostToDevice));
  d.ntiles = b.size();
  d.flops = 0;
  d.small = small;
  DMRG_REQUIRE(!small || b.size() % kOneWaves == 0, kErrState, "gemm: a small launch has whole workgroups of tiles");
  for (const GemmOne& t : b)
    if (t.m > 0) {
      DMRG_REQUIRE(t.m <= (small ? kOneSmall : kOneRows) && t.n <= (small ? one_small_cols(t.m) : kOneCols) && t.k > 0, kErrState,
                   "gemm: single-product tile out of range");
      d.flops += 2.0 * t.m * t.n * t.k;
      ++d.nsegs;
    }
}

void launch_gemm_f64(const DevGemm& d, hipStream_t stream, int role) {
  for (size_t off = 0; off < d.ntiles; off += (size_t)1 << 30) {
    const unsigned cnt = (unsigned)std::min<size_t>(d.ntiles - off, (size_t)1 << 30);
#define DMRG_ONE(SMALL, RAW) \
  hipLaunchKernelGGL((k_gemm_f64_one<1, SMALL, RAW>), dim3(SMALL ? cnt / kOneWaves : cnt), dim3(64 * kOneWaves), 0, stream, d.ones + off)
#define DMRG_KS(SMALL, RAW)                                                                             \
  hipLaunchKernelGGL((k_gemm_f64_ks<2, SMALL, RAW>), dim3(cnt), dim3(64 * kKsWaves), 0, stream, d.tiles + off, \
                     d.segs, d.shares)
    if (d.ones) {
      if (d.small) { if (d.raw) DMRG_ONE(true, true); else DMRG_ONE(true, false); }
      else { if (d.raw) DMRG_ONE(false, true); else DMRG_ONE(false, false); }
      continue;
    }
    if (d.ksplit) {
      if (d.small) { if (d.raw) DMRG_KS(true, true); else DMRG_KS(true, false); }
      else { if (d.raw) DMRG_KS(false, true); else DMRG_KS(false, false); }
      continue;
    }
#undef DMRG_ONE
#undef DMRG_KS
    launch_f64_tiles(role, d.tile, d.tile_n, d.lds, cnt, stream, d.tiles + off, d.segs);
  }
  DMRG_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
__global__ void k_scale(double* x, double a, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] *= a;
}
__global__ void k_axpy(double* y, double a, const double* x, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] += a * x[i];
}
__global__ void k_axpby(double* z, double a, const double* x, double b, const double* y,
                        int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    z[i] = a * x[i] + b * y[i];
}
__global__ void k_fill(double* x, double v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = v;
}

static unsigned grid_for(int64_t n) {
  int64_t g = (n + 255) / 256;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, 4096));
}

void launch_scale(double* x, double a, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_scale, dim3(grid_for(n)), dim3(256), 0, s, x, a, n);
  DMRG_HIP(hipGetLastError());
}
void launch_axpy(double* y, double a, const double* x, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_axpy, dim3(grid_for(n)), dim3(256), 0, s, y, a, x, n);
  DMRG_HIP(hipGetLastError());
}
void launch_axpby(double* z, double a, const double* x, double b, const double* y, int64_t n,
                  hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_axpby, dim3(grid_for(n)), dim3(256), 0, s, z, a, x, b, y, n);
  DMRG_HIP(hipGetLastError());
}
void launch_fill(double* x, double v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill, dim3(grid_for(n)), dim3(256), 0, s, x, v, n);
  DMRG_HIP(hipGetLastError());
}

// Deterministic two-pass dot products: block partials, then one block per row.
constexpr int kDotBlocks = 512;
__global__ __launch_bounds__(256) void k_multidot_partial(double* part, const double* X,
                                                          int64_t ldx, const double* y,
                                                          int64_t n) {
  __shared__ double red[256];
  const int j = blockIdx.y;
  const double* x = X + j * ldx;
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    acc += x[i] * y[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(int64_t)j * gridDim.x + blockIdx.x] = red[0];
}
__global__ __launch_bounds__(256) void k_reduce_rows(double* out, const double* part, int nb) {
  __shared__ double red[256];
  const int j = blockIdx.x;
  double acc = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) acc += part[(int64_t)j * nb + i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[j] = red[0];
}

void launch_multidot(double* out, const double* X, int64_t ldx, int nv, const double* y,
                     int64_t n, hipStream_t s) {
  if (nv <= 0) return;
  static thread_local DevBuf part;
  const size_t need = (size_t)nv * kDotBlocks * sizeof(double);
  if (part.bytes < need) {
    DMRG_HIP(hipStreamSynchronize(s));
    part.alloc(need);
  }
  int nb = (int)std::max<int64_t>(1, std::min<int64_t>(kDotBlocks, (n + 255) / 256));
  hipLaunchKernelGGL(k_multidot_partial, dim3(nb, nv), dim3(256), 0, s, part.as<double>(), X,
                     ldx, y, n);
  hipLaunchKernelGGL(k_reduce_rows, dim3(nv), dim3(256), 0, s, out, part.as<double>(), nb);
  DMRG_HIP(hipGetLastError());
}

__global__ void k_lincomb(double* y, const double* X, int64_t ldx, int nv, const double* c,
                          int64_t n, double alpha, double beta) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double acc = beta == 0.0 ? 0.0 : beta * y[i];
    for (int j = 0; j < nv; ++j) acc += (alpha * c[j]) * X[j * ldx + i];
    y[i] = acc;
  }
}
void launch_lincomb(double* y, const double* X, int64_t ldx, int nv, const double* c,
                    int64_t n, double beta, hipStream_t s, double alpha) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_lincomb, dim3(grid_for(n)), dim3(256), 0, s, y, X, ldx, nv, c, n, alpha, beta);
  DMRG_HIP(hipGetLastError());
}

__global__ void k_row_scatter_add(double* dst, const double* src, const int64_t* off, int64_t n) {
  const int r = blockIdx.y;
  double* d = dst + off[r];
  const double* x = src + (int64_t)r * n;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    d[i] += x[i];
}
void launch_row_scatter_add(double* dst, const double* src, const int64_t* dst_off, int nrows,
                            int64_t n, hipStream_t s) {
  if (nrows <= 0 || n <= 0) return;
  unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 64));
  hipLaunchKernelGGL(k_row_scatter_add, dim3(gx, nrows), dim3(256), 0, s, dst, src, dst_off, n);
  DMRG_HIP(hipGetLastError());
}

__global__ void k_copy_tasks(const CopyTask* tasks, int transpose) {
  const CopyTask t = tasks[blockIdx.x];
  const int64_t n = (int64_t)t.rows * t.cols;
  for (int64_t e = threadIdx.x; e < n; e += blockDim.x) {
    const int r = (int)(e / t.cols), c = (int)(e % t.cols);
    if (transpose) t.dst[(int64_t)c * t.dld + r] = t.src[(int64_t)r * t.sld + c];
    else t.dst[(int64_t)r * t.dld + c] = t.src[(int64_t)r * t.sld + c];
  }
}
void launch_copy_tasks(const CopyTask* tasks, int ntasks, bool transpose, hipStream_t s) {
  if (ntasks <= 0) return;
  hipLaunchKernelGGL(k_copy_tasks, dim3(ntasks), dim3(256), 0, s, tasks, (int)transpose);
  DMRG_HIP(hipGetLastError());
}

// psi block piece into the padded copy and its transpose: a piece of at most
// kPackTile x kPackTile is read once, row by row, and leaves twice, as rows
// and, through LDS, as columns, both in whole cache lines.  The BF16 planes of
// both copies and the zeros that the pinned pairs add to leave with it: small
// sigmas are bound by their launches (12 orbitals D = 100, BF16x3 with nine
// launches 174 us, 168 with the split and the fill in this one).
constexpr int kPackZeros = 4096;  // doubles that a workgroup past the tasks clears
template <bool BF>
__global__ __launch_bounds__(256) void k_pack_psi(const PackTask* __restrict__ tasks, int ntasks,
                                                  const double* __restrict__ psi, const PackMore more) {
  if ((int)blockIdx.x >= ntasks) {
    const int64_t z0 = (int64_t)((int)blockIdx.x - ntasks) * kPackZeros;
    for (int64_t i = z0 + threadIdx.x; i < min(z0 + kPackZeros, more.nz); i += 256) more.z[i] = 0.0;
    return;
  }
  __shared__ double sm[kPackTile][kPackTile + 1];
  const PackTask t = tasks[blockIdx.x];
  auto split = [](uint16_t* bf, int64_t n, int64_t at, double x) {
    const uint16_t hi = f32_to_bf16_rn((float)x);
    bf[at] = hi;
    bf[at + n] = f32_to_bf16_rn((float)(x - (double)bf16_to_f32(hi)));
  };
  const int c = threadIdx.x % kPackTile;
  for (int r = threadIdx.x / kPackTile; r < t.rows; r += 256 / kPackTile)
    if (c < t.cols) {
      const double x = psi[t.src + (int64_t)r * t.sld + c];
      double* d = t.dst + (int64_t)r * t.dld + c;
      *d = x;
      if (BF) split(more.bf, more.n, d - more.p, x);
      sm[r][c] = x;
    }
  if (!t.dstT) return;
  __syncthreads();
  const int r = threadIdx.x % kPackTile;
  for (int q = threadIdx.x / kPackTile; q < t.cols; q += 256 / kPackTile)
    if (r < t.rows) {
      double* d = t.dstT + (int64_t)q * t.tld + r;
      *d = sm[r][q];
      if (BF) split(more.bfT, more.nT, d - more.t, sm[r][q]);
    }
}
void launch_pack_psi(const PackTask* tasks, int ntasks, const double* psi, hipStream_t s, const PackMore& more) {
  const int64_t blocks = ntasks + (more.nz + kPackZeros - 1) / kPackZeros;
  if (blocks <= 0) return;
  if (more.bf) hipLaunchKernelGGL(k_pack_psi<true>, dim3((unsigned)blocks), dim3(256), 0, s, tasks, ntasks, psi, more);
  else hipLaunchKernelGGL(k_pack_psi<false>, dim3((unsigned)blocks), dim3(256), 0, s, tasks, ntasks, psi, more);
  DMRG_HIP(hipGetLastError());
}

// sigma block piece out of the padded copy, with the partial sums of its
// output problem added in order.
__global__ __launch_bounds__(256) void k_unpack_sigma(const SumTask* __restrict__ tasks, double* __restrict__ sigma) {
  const SumTask t = tasks[blockIdx.x];
  for (int r = threadIdx.x >> 5; r < t.rows; r += 8)
    for (int c = threadIdx.x & 31; c < t.cols; c += 32) {
      const int64_t e = (int64_t)r * t.sld + c;
      double x = t.nparts < 0 ? 0.0 : t.src[e];
      const double* p = t.part + e;
      int j = 0;
      for (; j + 4 <= t.nparts; j += 4) {  // four loads in flight, added in order
        const double p0 = p[j * t.stride], p1 = p[(j + 1) * t.stride], p2 = p[(j + 2) * t.stride],
                     p3 = p[(j + 3) * t.stride];
        x = (((x + p0) + p1) + p2) + p3;
      }
      for (; j < t.nparts; ++j) x += p[j * t.stride];
      sigma[t.dst + (int64_t)r * t.dld + c] = x;
    }
}
void launch_unpack_sigma(const SumTask* tasks, int ntasks, double* sigma, hipStream_t s) {
  if (ntasks <= 0) return;
  hipLaunchKernelGGL(k_unpack_sigma, dim3(ntasks), dim3(256), 0, s, tasks, sigma);
  DMRG_HIP(hipGetLastError());
}

// ---- Davidson helpers --------------------------------------------------------
__global__ void k_extract_diag(const DiagTask* tasks) {
  const DiagTask t = tasks[blockIdx.x];
  for (int i = threadIdx.x; i < t.d; i += blockDim.x) t.dst[i] = t.src[(int64_t)i * (t.ld + 1)];
}
void launch_extract_diag(const DiagTask* tasks, int ntasks, hipStream_t s) {
  for (int off = 0; off < ntasks; off += 1 << 30) {
    const int cnt = std::min(ntasks - off, 1 << 30);
    hipLaunchKernelGGL(k_extract_diag, dim3(cnt), dim3(64), 0, s, tasks + off);
  }
  DMRG_HIP(hipGetLastError());
}

// diag[row][col] = sum_p yd[p][n(row)] * Ld[p][aL(row)] * Zd[p][offR + col]
__global__ __launch_bounds__(256) void k_heff_diag(double* out, int64_t rows, int dr,
                                                   const int64_t* rowinfo, int64_t offR,
                                                   int npairs, const double* yd,
                                                   const double* Ld, int64_t DL,
                                                   const double* Zd, int64_t DR) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= rows * dr) return;
  const int64_t row = e / dr;
  const int col = (int)(e % dr);
  const int64_t aL = rowinfo[2 * row];
  const int n = (int)rowinfo[2 * row + 1];
  double acc = 0.0;
  for (int p = 0; p < npairs; ++p)
    acc += yd[p * 16 + n] * Ld[p * DL + aL] * Zd[p * DR + offR + col];
  out[e] = acc;
}
void launch_heff_diag(double* out, int64_t rows, int dr, const int64_t* rowinfo, int64_t offR,
                      int npairs, const double* yd, const double* Ld, int64_t DL,
                      const double* Zd, int64_t DR, hipStream_t s) {
  const int64_t n = rows * dr;
  if (n <= 0) return;
  hipLaunchKernelGGL(k_heff_diag, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, rows, dr,
                     rowinfo, offR, npairs, yd, Ld, DL, Zd, DR);
  DMRG_HIP(hipGetLastError());
}

// ---- Davidson steps whose coefficients stay on the device -----------------
// (a step of 14 orbitals D = 256, n = 67 000, spent 0.25 of 0.6 ms on sigma:
// the rest was waits for coefficients that went to the host and back)

// u = V y, w = W y, r = w - theta u
__global__ __launch_bounds__(256) void k_ritz(double* u, double* w, double* r, const double* V, const double* W,
                                              int64_t n, int k, const double* y, const double* theta) {
  const double th = *theta;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double a = 0.0, b = 0.0;
    for (int j = 0; j < k; ++j) {
      a += y[j] * V[j * n + i];
      b += y[j] * W[j * n + i];
    }
    u[i] = a;
    w[i] = b;
    r[i] = b + -th * a;
  }
}
void launch_ritz(double* u, double* w, double* r, const double* V, const double* W, int64_t n, int k, const double* y,
                 const double* theta, hipStream_t s) {
  hipLaunchKernelGGL(k_ritz, dim3(grid_for(n)), dim3(256), 0, s, u, w, r, V, W, n, k, y, theta);
  DMRG_HIP(hipGetLastError());
}

// t -= (num / den) x where den is not tiny (num = c[0], den = c[1])
__global__ void k_olsen(double* t, const double* x, const double* c, int64_t n) {
  if (!(fabs(c[1]) > 1e-300)) return;
  const double a = -c[0] / c[1];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    t[i] += a * x[i];
}
void launch_olsen(double* t, const double* x, const double* c, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_olsen, dim3(grid_for(n)), dim3(256), 0, s, t, x, c, n);
  DMRG_HIP(hipGetLastError());
}

__global__ void k_scale_to(double* y, double a, const double* x, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = a * x[i];
}
void launch_scale_to(double* y, double a, const double* x, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_to, dim3(grid_for(n)), dim3(256), 0, s, y, a, x, n);
  DMRG_HIP(hipGetLastError());
}

// Column c of the symmetric subspace matrix G (kmax x kmax) from h, and its
// leading (c + 1) x (c + 1) part, packed, into A.  One workgroup.
__global__ __launch_bounds__(256) void k_subspace(double* G, int kmax, const double* h, int c, double* A) {
  for (int i = threadIdx.x; i <= c; i += blockDim.x) G[i * kmax + c] = G[c * kmax + i] = h[i];
  __syncthreads();
  const int k = c + 1;
  for (int e = threadIdx.x; e < k * k; e += blockDim.x) A[e] = G[(e / k) * kmax + e % k];
}
void launch_subspace(double* G, int kmax, const double* h, int c, double* A, hipStream_t s) {
  hipLaunchKernelGGL(k_subspace, dim3(1), dim3(256), 0, s, G, kmax, h, c, A);
  DMRG_HIP(hipGetLastError());
}

// out = min of x (n >= 1).  One workgroup of 1024.
__global__ __launch_bounds__(1024) void k_min(double* out, const double* x, int64_t n) {
  __shared__ double red[1024];
  double m = x[0];
  for (int64_t i = threadIdx.x; i < n; i += 1024) m = x[i] < m ? x[i] : m;
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w && red[threadIdx.x + w] < red[threadIdx.x]) red[threadIdx.x] = red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}
// out = min of x in two passes over part (at least kDotBlocks doubles)
__global__ __launch_bounds__(256) void k_min_partial(double* part, const double* x, int64_t n) {
  __shared__ double red[256];
  double m = x[0];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    m = x[i] < m ? x[i] : m;
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w && red[threadIdx.x + w] < red[threadIdx.x]) red[threadIdx.x] = red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}
void launch_min(double* out, double* part, const double* x, int64_t n, hipStream_t s) {
  const int nb = (int)std::max<int64_t>(1, std::min<int64_t>(kDotBlocks, (n + 255) / 256));
  hipLaunchKernelGGL(k_min_partial, dim3(nb), dim3(256), 0, s, part, x, n);
  hipLaunchKernelGGL(k_min, dim3(1), dim3(1024), 0, s, out, part, (int64_t)nb);
  DMRG_HIP(hipGetLastError());
}

// t = r / (theta - d), the denominator clamped to |.| >= 1e-8 keeping its sign
__global__ void k_precondition(double* t, const double* r, const double* d, double theta,
                               int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double den = theta - d[i];
    if (fabs(den) < 1e-8) den = den < 0 ? -1e-8 : 1e-8;
    t[i] = r[i] / den;
  }
}
void launch_precondition(double* t, const double* r, const double* d, double theta, int64_t n,
                         hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_precondition, dim3(grid_for(n)), dim3(256), 0, s, t, r, d, theta, n);
  DMRG_HIP(hipGetLastError());
}

}  // namespace dmrg
