// Ozaki-scheme FP64 emulation on gfx950 INT8 MFMA (see gemm_oz.h).
//
// k_slice_oz: one workgroup per 64 rows of an operand.  8 to 64 lanes take a
// row, four entries each: the row maximum (reduction over those lanes) gives
// the exponent e with |x| < (127/128) 2^e, so that every rounded
// X = round(x 2^(p - e)) has a kappa-digit signed base-256 expansion; the
// digits are written as kappa int8 planes (four entries a lane, one 32-bit
// store per plane, coalesced along k).  Bound by memory latency: short rows
// need few lanes each so that the loads of many rows are in flight (operands
// of about 30 x 30, 95012 of them at 16 orbitals D = 512: 1650 -> 344 us
// against a whole wave per row; psi, large operands: 208 -> 11 us by 64-row
// tasks).
//
// k_gemm_oz: the task model of the other grouped GEMMs (one workgroup per
// 64 x 64 output tile, a list of segments), four waves as 2 x 2 with 32 x 32
// each in MFMA 16x16x64 INT8 blocks.  A slab holds 64 k entries of every
// digit plane of both operands (kappa (64 + 64) rows of 64 bytes), loaded
// straight into LDS (global_load_lds, 16 bytes a lane, XOR-swizzled rows).
// Per slab and 16 x 16 block the kappa (kappa + 1) / 2 digit products with
// s + t >= kappa - 1 accumulate in INT32, one accumulator per weight s + t;
// at the end of a segment the weights are combined in FP64 (Horner in 256),
// scaled by 2^(e_i + f_j - 2p) and the segment scale, and added to an FP64
// register accumulator, which is written (or added) once per tile.
// A segment is mostly one slab, so a tile is a chain of load, multiply,
// combine.  One slab of LDS (48 KB with six digits) and 228 registers leave
// two workgroups on a CU, which fill each other's waits: the fragments go to
// registers, the buffer is free again before the larger part of the products,
// and the next slab and its exponents travel under them (three slabs of LDS
// and one workgroup a CU: stage 1 1587 us, now 685; stage 2, which also ran
// its 304 lists uncut, 3665 us, now 821; 16 orbitals D = 512).  With seven
// digits the two workgroups' 256 registers spill six (20 bytes a lane), which
// costs less than the second workgroup gives: a whole sigma, before and now,
// ms, with 3, 6 and 7 digits: 16 orbitals D = 512 4.35 -> 1.13, 7.21 -> 1.92,
// 21.2 -> 2.36; 12 orbitals D = 1500 7.09 -> 2.69, 14.1 -> 4.68, 42.9 -> 5.73.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gemm_oz.h"

namespace dmrg {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int oz_swz(int row) { return (row >> 1) & 3; }
__device__ __forceinline__ i32x4 oz_frag(const int8_t* part, int row, int q) {
  return *reinterpret_cast<const i32x4*>(part + row * 64 + 16 * (q ^ oz_swz(row)));
}

// Digits of four consecutive entries (X: rounded integers) as one 32-bit
// store per plane.
__device__ __forceinline__ void oz_store_digits(int8_t* dst, int64_t plane, int kappa, int64_t X[4]) {
  for (int s = 0; s < kappa; ++s) {
    uint32_t w = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t d = ((X[u] + 128) & 255) - 128;
      w |= (uint32_t)(uint8_t)(int8_t)d << (8 * u);
      X[u] = (X[u] - d) >> 8;
    }
    *reinterpret_cast<uint32_t*>(dst + (int64_t)s * plane) = w;
  }
}

// G lanes take a row, four consecutive entries each (rows of more than 4 G
// entries: 4 G at a time, read twice), so a wave holds 64 / G rows at once.
template <int G>
__device__ __forceinline__ void oz_slice_rows(const SliceOp& op, int8_t* arena, int32_t* exps, int kappa) {
  const int P = 8 * kappa - 1;
  const int k0 = 4 * (threadIdx.x & (G - 1));
  const bool vec = !op.colmajor && op.ld % 2 == 0 && (reinterpret_cast<uintptr_t>(op.src) & 15) == 0;
  auto load4 = [&](int i, int kk, double v[4]) {
    if (vec && kk + 4 <= op.k) {
      const double2* p = reinterpret_cast<const double2*>(op.src + (int64_t)i * op.ld + kk);
      const double2 x = p[0], y = p[1];
      v[0] = x.x; v[1] = x.y; v[2] = y.x; v[3] = y.y;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u] = kk + u >= op.k   ? 0.0
               : op.colmajor ? op.src[(int64_t)(kk + u) * op.ld + i]
                             : op.src[(int64_t)i * op.ld + kk + u];
    }
  };
  for (int i = (int)threadIdx.x / G; i < op.rows; i += 256 / G) {
    double v[4];
    load4(i, k0, v);
    double mx = fmax(fmax(fabs(v[0]), fabs(v[1])), fmax(fabs(v[2]), fabs(v[3])));
    if constexpr (G == 64)
      for (int kk = k0 + 4 * G; kk < op.k; kk += 4 * G) {
        double z[4];
        load4(i, kk, z);
        mx = fmax(mx, fmax(fmax(fabs(z[0]), fabs(z[1])), fmax(fabs(z[2]), fabs(z[3]))));
      }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    // |x| <= mx < (127/128) 2^e keeps X inside the kappa-digit range
    const int e = mx > 0.0 ? ilogb(mx * (128.0 / 127.0)) + 1 : 0;
    if (k0 == 0) exps[op.exp + i] = e;
    int8_t* row = arena + op.dst + (int64_t)i * op.kp;
    for (int kk = k0; kk < op.kp; kk += 4 * G) {
      if (G == 64 && kk != k0) load4(i, kk, v);
      int64_t X[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) X[u] = (int64_t)rint(ldexp(v[u], P - e));
      oz_store_digits(row + kk, op.plane, kappa, X);
    }
  }
}

__global__ __launch_bounds__(256) void k_slice_oz(const SliceOp* __restrict__ ops, int8_t* arena, int32_t* exps,
                                                  int kappa) {
  const SliceOp op = ops[blockIdx.x];
  if (op.kp <= 32) oz_slice_rows<8>(op, arena, exps, kappa);
  else if (op.kp <= 64) oz_slice_rows<16>(op, arena, exps, kappa);
  else if (op.kp <= 128) oz_slice_rows<32>(op, arena, exps, kappa);
  else oz_slice_rows<64>(op, arena, exps, kappa);
}

template <int KAPPA>
__global__ __launch_bounds__(256, 2) void k_gemm_oz(const GemmTileB* __restrict__ tiles,
                                                    const GemmSegO* __restrict__ segs) {
  constexpr int P = 8 * KAPPA - 1;
  constexpr int PLANE = kOzTile * kOzBK;  // bytes of one digit plane of one operand's slab
  constexpr int NEXT = KAPPA / 2;         // digits of A multiplied before the next slab's loads start
  __shared__ __attribute__((aligned(16))) int8_t smem[2 * KAPPA * PLANE];
  int8_t* const slab = smem;
  __shared__ int32_t sexp[2 * kOzTile];  // row exponents of A and B of the current segment
  const GemmTileB t = tiles[blockIdx.x];
  if (t.m <= 0) return;  // padding tile of an XCD-ordered launch
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int lr = lane & 15, lk = lane >> 4;
  const bool idle = __builtin_amdgcn_readfirstlane((int)(wm >= t.m || wn >= t.n)) != 0;
  i32x4 acc[KAPPA][2][2];  // by weight s + t - (KAPPA - 1)
  double acc64[2][2][4];
#pragma unroll
  for (int w = 0; w < KAPPA; ++w)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[w][a][b] = i32x4{0, 0, 0, 0};
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc64[a][b][v] = 0.0;

  // Loads: wave w takes rows 16 w .. 16 w + 15 of every digit plane (four
  // 16-byte chunks a row, swizzled).  Rows past the tile repeat its last row
  // (their products are not stored); chunks past the segment repeat the
  // slab's first chunk, and the fragments of A set them to zero.
  const int lrow = 16 * wave + (lane >> 2);
  const int chunk = 16 * ((lane & 3) ^ oz_swz(lrow));
  const int arow = min(lrow, t.m - 1), brow = min(lrow, t.n - 1);
  const int erow = wave == 0 ? min(lane, t.m - 1) : min(lane, t.n - 1);
  int ps = t.seg_begin, pk0 = 0, cs = ps, ck0 = 0;
  GemmSegO pg = segs[ps];
  int ckpad = oz_kp(pg.k);
  double alpha = pg.alpha;
  auto load_rows = [](const int8_t* src, int8_t* dst) { __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0); };
  auto produce = [&]() {
    const int kpad = oz_kp(pg.k);
    const int c = pk0 + chunk < kpad ? chunk : 0;
    const int8_t* pa = pg.a + (int64_t)t.row0 * pg.lda + pk0;
    const int8_t* pb = pg.b + (int64_t)t.col0 * pg.ldb + pk0;
    const uint32_t oa = (uint32_t)(arow * pg.lda + c), ob = (uint32_t)(brow * pg.ldb + c);
#pragma unroll
    for (int j = 0; j < KAPPA; ++j)
      load_rows(pa + j * pg.a_plane + oa, slab + j * PLANE + 1024 * wave);
#pragma unroll
    for (int j = 0; j < KAPPA; ++j)
      load_rows(pb + j * pg.b_plane + ob, slab + (KAPPA + j) * PLANE + 1024 * wave);
    if (pk0 == 0 && wave < 2)  // a new segment: its exponents, 64 rows of A (wave 0) and of B (wave 1)
      __builtin_amdgcn_global_load_lds((wave == 0 ? pg.ea + t.row0 : pg.eb + t.col0) + erow, sexp + kOzTile * wave, 4, 0, 0);
    pk0 += kOzBK;
    if (pk0 >= kpad) {
      pk0 = 0;
      if (++ps < t.seg_end) pg = segs[ps];
    }
  };
  produce();
  while (true) {
    // the slab has landed in every wave's part of LDS
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const bool last = ck0 + kOzBK >= ckpad;  // the segment's last slab
    const bool dead = ck0 + 16 * lk >= ckpad;
    i32x4 bf[KAPPA][2], af[KAPPA][2];
    int ea[2][4], eb[2];
    auto mul = [&](int s) {
#pragma unroll
      for (int u = KAPPA - 1 - s; u < KAPPA; ++u)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[s + u - (KAPPA - 1)][a][b] =
                __builtin_amdgcn_mfma_i32_16x16x64_i8(af[s][a], bf[u][b], acc[s + u - (KAPPA - 1)][a][b], 0, 0, 0);
    };
    auto read_a = [&](int s) {
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        af[s][a] = oz_frag(slab + s * PLANE, wm + 16 * a + lr, lk);
        if (dead) af[s][a] = i32x4{0, 0, 0, 0};
      }
    };
    if (!idle) {
#pragma unroll
      for (int s = 0; s < KAPPA; ++s)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          bf[KAPPA - 1 - s][b] = oz_frag(slab + (2 * KAPPA - 1 - s) * PLANE, wn + 16 * b + lr, lk);
#pragma unroll
      for (int s = 0; s < NEXT; ++s) {
        read_a(s);
        mul(s);
      }
#pragma unroll
      for (int s = NEXT; s < KAPPA; ++s) read_a(s);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) ea[a][v] = sexp[wm + 16 * a + 4 * lk + v];
#pragma unroll
      for (int b = 0; b < 2; ++b) eb[b] = sexp[kOzTile + wn + 16 * b + lr];
    }
    const bool more = ps < t.seg_end;
    if (more) {
      // every wave has its fragments in registers (lgkmcnt(0)): LDS is free,
      // and the next slab travels under the larger part of the products
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      produce();
    }
    if (!idle) {
#pragma unroll
      for (int s = NEXT; s < KAPPA; ++s) mul(s);
      if (last) {
        // segment finished: combine the weights in FP64 with the row scales
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              double x = 0.0;
#pragma unroll
              for (int w = KAPPA - 1; w >= 0; --w) x = x * 256.0 + (double)acc[w][a][b][v];
              acc64[a][b][v] += alpha * ldexp(x, ea[a][v] + eb[b] - 2 * P + 8 * (KAPPA - 1));
            }
#pragma unroll
        for (int w = 0; w < KAPPA; ++w)
#pragma unroll
          for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[w][a][b] = i32x4{0, 0, 0, 0};
      }
    }
    if (!more) break;
    ck0 += kOzBK;
    if (last) {
      ck0 = 0;
      ++cs;
      ckpad = oz_kp(segs[cs].k);
      alpha = segs[cs].alpha;
    }
  }
  if (idle) return;
  double* C = static_cast<double*>(t.c);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = wm + 16 * a + 4 * lk + v;
        const int j = wn + 16 * b + lr;
        if (i >= t.m || j >= t.n) continue;
        const int64_t idx = ((int64_t)t.row0 + i) * t.ldc + (t.col0 + j);
        C[idx] = t.beta ? C[idx] + acc64[a][b][v] : acc64[a][b][v];
      }
}

template __global__ void k_gemm_oz<3>(const GemmTileB*, const GemmSegO*);
template __global__ void k_gemm_oz<4>(const GemmTileB*, const GemmSegO*);
template __global__ void k_gemm_oz<5>(const GemmTileB*, const GemmSegO*);
template __global__ void k_gemm_oz<6>(const GemmTileB*, const GemmSegO*);
template __global__ void k_gemm_oz<7>(const GemmTileB*, const GemmSegO*);

}  // namespace

void launch_slice_oz(const SliceOp* ops, int nops, int64_t rows, int8_t* arena, int32_t* exps, int kappa,
                     hipStream_t s) {
  if (rows <= 0 || nops <= 0) return;
  DMRG_REQUIRE(kappa >= kOzMinKappa && kappa <= kOzMaxKappa, kErrInvalidArg, "slice_oz: kappa out of range");
  hipLaunchKernelGGL(k_slice_oz, dim3((unsigned)nops), dim3(256), 0, s, ops, arena, exps, kappa);
  DMRG_HIP(hipGetLastError());
}

void upload_gemm_oz(const GemmBatchO& b, int kappa, DevGemmO& d) {
  // the INT32 accumulator of one weight sums up to kappa digit products of
  // one segment: kappa * k * 2^14 < 2^31
  for (const GemmSegO& g : b.segs)
    DMRG_REQUIRE((int64_t)kappa * g.k * 16384 < ((int64_t)1 << 31), kErrShape,
                 "gemm_oz: segment k too large for exact INT32 accumulation");
  const size_t sb = b.segs.size() * sizeof(GemmSegO);
  const size_t tb = b.tiles.size() * sizeof(GemmTileB);
  const size_t sba = ((sb + 255) / 256) * 256;
  d.buf.alloc(sba + tb + 256);
  d.segs = reinterpret_cast<GemmSegO*>(d.buf.as<char>());
  d.tiles = reinterpret_cast<GemmTileB*>(d.buf.as<char>() + sba);
  if (sb) DMRG_HIP(hipMemcpy(d.segs, b.segs.data(), sb, hipMemcpyHostToDevice));
  if (tb) DMRG_HIP(hipMemcpy(d.tiles, b.tiles.data(), tb, hipMemcpyHostToDevice));
  d.ntiles = b.tiles.size();
  d.nsegs = b.segs.size();
}

void launch_gemm_oz(const DevGemmO& d, int kappa, hipStream_t s) {
  for (size_t off = 0; off < d.ntiles; off += (size_t)1 << 30) {
    const unsigned cnt = (unsigned)std::min<size_t>(d.ntiles - off, (size_t)1 << 30);
    const GemmTileB* tl = d.tiles + off;
    switch (kappa) {
      case 3: hipLaunchKernelGGL(k_gemm_oz<3>, dim3(cnt), dim3(256), 0, s, tl, d.segs); break;
      case 4: hipLaunchKernelGGL(k_gemm_oz<4>, dim3(cnt), dim3(256), 0, s, tl, d.segs); break;
      case 5: hipLaunchKernelGGL(k_gemm_oz<5>, dim3(cnt), dim3(256), 0, s, tl, d.segs); break;
      case 6: hipLaunchKernelGGL(k_gemm_oz<6>, dim3(cnt), dim3(256), 0, s, tl, d.segs); break;
      case 7: hipLaunchKernelGGL(k_gemm_oz<7>, dim3(cnt), dim3(256), 0, s, tl, d.segs); break;
      default: DMRG_REQUIRE(false, kErrInvalidArg, "gemm_oz: kappa out of range");
    }
  }
  DMRG_HIP(hipGetLastError());
}

}  // namespace dmrg
