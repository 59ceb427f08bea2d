// Per-frequency-bin complex contraction (arXiv:1601.06815, Introduction and
// Section 2: the Hadamard product of block and kernel spectra, summed over the
// C channels of the layer; Section 3.2 for the two backward products).
//
// For every bin f (the unique bins only, see unique_bin) the three passes are
// complex matrix products:
//   forward          Yhat[f]  (K x BP) = What[f]^T   (K x C)  * Xhat[f] (C x BP)
//   backward_data    dXhat[f] (C x BP) = conj What[f] (C x K)  * Ghat[f] (K x BP)
//   backward_filter  dWhat[f] (C x K)  = conj Xhat[f] (C x BP) * Ghat[f]^T (BP x K)
// and, to compose two stacked layers in the frequency domain (Conclusion),
//   W12hat[f] (C x K) = W1hat[f] (C x J) * W2hat[f] (J x K).
//
// Two implementations, both staging 16-deep slices of the reduction for one
// output tile through LDS, with the next slice loaded into registers while
// the current one is consumed:
//  * vector ALU: real and imaginary planes, 64 x 64 complex tile per 256-lane
//    workgroup, 4 x 4 complex accumulators per lane, four real multiply-adds
//    per complex one;
//  * bf16 matrix cores (v_mfma_f32_16x16x32_bf16) on operands split exactly
//    into three bf16 pieces each, with fp32 accumulation: 16 x 64 to 128 x 128
//    complex tiles per workgroup, persistent workgroups walking the tiles in
//    XCD-local rounds, operands read through buffer resources. Results of
//    values that three pieces do not hold (below 2^-110, above 3.396e38) are
//    taken again in fp32 multiply-adds.
#include <algorithm>
#include <atomic>

#include "buffer_io.hpp"
#include "mfma_tiles.hpp"
#include "oaa_internal.hpp"
#include "tile_common.hpp"

namespace oaa {

namespace {

constexpr int kThreads = 256;
constexpr int kKC = kMfmaSlice;  // reduction depth of one LDS slice

// A ROWS x kKC slice of an operand whose element (row, k) is stored at
// X[k*ld + row] (ROW_CONTIG) or X[row*ld + k]; loads are coalesced along the
// contiguous index. Out-of-range elements read a valid clamped address and
// are replaced by zero.
template <bool ROW_CONTIG, int ROWS>
struct Slice {
  static constexpr int PER = ROWS * kKC / kThreads;
  float2 v[PER];

  __device__ __forceinline__ static void coords(int e, int& rl, int& kl) {
    if (ROW_CONTIG) {
      rl = e % ROWS;
      kl = e / ROWS;
    } else {
      kl = e % kKC;
      rl = e / kKC;
    }
  }

  __device__ __forceinline__ void load(const float2* X, long ld, int r0, int nrows, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      int rl, kl;
      coords(int(threadIdx.x) + kThreads * i, rl, kl);
      const int r = r0 + rl, k = k0 + kl;
      const bool ok = r < nrows && k < kend;
      const int rc = ok ? r : r0, kc = ok ? k : k0;
      const float2 t = ROW_CONTIG ? X[size_t(kc) * ld + rc] : X[size_t(rc) * ld + kc];
      v[i] = ok ? t : make_float2(0.f, 0.f);
    }
  }

  template <int LD>
  __device__ __forceinline__ void store(float (*re)[LD], float (*im)[LD], bool conj) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      int rl, kl;
      coords(int(threadIdx.x) + kThreads * i, rl, kl);
      re[kl][rl] = v[i].x;
      im[kl][rl] = conj ? -v[i].y : v[i].y;
    }
  }
};

struct TileCoords {
  int f, split, m0, n0, k_begin, k_end;
};

template <int TM, int TN>
__device__ __forceinline__ TileCoords tile_coords(const GemmParams& p) {
  TileCoords t;
  t.f = unique_bin(blockIdx.z, p.L);
  t.split = blockIdx.y;
  const int tiles_n = (p.N + TN - 1) / TN;
  t.m0 = (blockIdx.x / tiles_n) * TM;
  t.n0 = (blockIdx.x % tiles_n) * TN;
  t.k_begin = t.split * p.kchunk;
  t.k_end = min(p.Kr, t.k_begin + p.kchunk);
  return t;
}

// ---------------------------------------------------------------------------
// vector-ALU implementation

constexpr int kVM = 64, kVN = 64;

template <bool AT, bool AC, bool BT, bool BC>
__global__ void __launch_bounds__(kThreads) cgemm_valu_kernel(GemmParams p) {
  __shared__ float Asr[kKC][kVM + 4], Asi[kKC][kVM + 4];
  __shared__ float Bsr[kKC][kVN + 4], Bsi[kKC][kVN + 4];
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const TileCoords tc = tile_coords<kVM, kVN>(p);
  const float2* A = p.A + size_t(tc.f) * p.a_fstride;
  const float2* B = p.B + size_t(tc.f) * p.b_fstride;

  float accr[4][4], acci[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) accr[i][j] = acci[i][j] = 0.f;

  Slice<AT, kVM> sa;
  Slice<!BT, kVN> sb;
  sa.load(A, p.lda, tc.m0, p.M, tc.k_begin, tc.k_end);
  sb.load(B, p.ldb, tc.n0, p.N, tc.k_begin, tc.k_end);
  for (int k0 = tc.k_begin; k0 < tc.k_end; k0 += kKC) {
    sa.template store<kVM + 4>(Asr, Asi, AC);
    sb.template store<kVN + 4>(Bsr, Bsi, BC);
    __syncthreads();
    if (k0 + kKC < tc.k_end) {
      sa.load(A, p.lda, tc.m0, p.M, k0 + kKC, tc.k_end);
      sb.load(B, p.ldb, tc.n0, p.N, k0 + kKC, tc.k_end);
    }
#pragma unroll
    for (int kk = 0; kk < kKC; ++kk) {
      float ar[4], ai[4], br[4], bi[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ar[i] = Asr[kk][ty + 16 * i];
        ai[i] = Asi[kk][ty + 16 * i];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        br[j] = Bsr[kk][tx + 16 * j];
        bi[j] = Bsi[kk][tx + 16 * j];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          accr[i][j] = __builtin_fmaf(ar[i], br[j], accr[i][j]);
          accr[i][j] = __builtin_fmaf(-ai[i], bi[j], accr[i][j]);
          acci[i][j] = __builtin_fmaf(ar[i], bi[j], acci[i][j]);
          acci[i][j] = __builtin_fmaf(ai[i], br[j], acci[i][j]);
        }
    }
    __syncthreads();
  }

  float2* Cm = p.C + size_t(tc.f) * p.c_fstride + size_t(tc.split) * p.c_sstride;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = tc.m0 + ty + 16 * i;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int nn = tc.n0 + tx + 16 * j;
      if (m < p.M && nn < p.N) Cm[size_t(m) * p.ldc + nn] = make_float2(accr[i][j], acci[i][j]);
    }
  }
}

// ---------------------------------------------------------------------------
// matrix-core implementation

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A complex value as three complex bf16 pieces, each packed (re low, im
// high): x = p0 + p1 + p2 exactly for components of 2^-110 to 3.396e38, since
// each rounding to nearest leaves a remainder of at most 16 and then 8
// significant bits of the 24, none below bf16's smallest number, 2^-133. Of a
// smaller component the last remainder may have bits below that; they are in
// its low 16 bits, which are or-ed to `lost`. A larger one rounds to infinity,
// and the remainder, infinity minus infinity in the end, to NaN.
__device__ __forceinline__ void split3(float2 x, unsigned& p0, unsigned& p1, unsigned& p2, unsigned& lost) {
  auto pack = [](float a, float b) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
  };
  auto lo = [](unsigned u) { return __builtin_bit_cast(float, u << 16); };
  auto hi = [](unsigned u) { return __builtin_bit_cast(float, u & 0xffff0000u); };
  p0 = pack(x.x, x.y);
  const float r1 = x.x - lo(p0), i1 = x.y - hi(p0);
  p1 = pack(r1, i1);
  const float r2 = r1 - lo(p1), i2 = i1 - hi(p1);
  p2 = pack(r2, i2);
  lost |= __builtin_bit_cast(unsigned, r2) | __builtin_bit_cast(unsigned, i2);
}

// LDS image of an operand's ROWS x kKC slice, one per piece: rows of four
// 16-byte quads, quad q holding reduction indices 4q .. 4q + 3 as packed
// complex pieces, stored at quad q ^ ((row / 2) % 4) ^ ((row / 8) % 2) of the row. The 16
// lanes that read one quad of 16 consecutive rows, and the lanes that write
// it, then fall on all 64 banks.
__device__ __forceinline__ constexpr int quad_at(int row, int q) {
  return row * 4 + (q ^ ((row >> 1) & 3) ^ ((row >> 3) & 1));
}

// One operand's ROWS x kKC slices, read through a buffer resource over one
// bin's matrix; element (row, k) is at k*ld + row (ROW_CONTIG) or row*ld + k.
// A task is a quad of one row: four loads, split into pieces and written to
// LDS as three quads. Lanes run along the rows (ROW_CONTIG) or along the
// four quads of a row, so that loads are coalesced. Elements outside the
// matrix or past the reduction bound get an offset beyond the resource, which
// the hardware reads as zero. Lane FIRST takes the first task, so that two
// small operands are staged by different waves.
// LONG: rows of any length that fits (ROW_CONTIG), past the 2^25 elements from
// which offsets of 16 of them, also those past a short reduction, wrap.
template <bool ROW_CONTIG, int ROWS, int THREADS, int FIRST, bool LONG>
struct Operand {
  static constexpr int TASKS = ROWS * 4, PER = (TASKS + THREADS - 1) / THREADS;
  static constexpr bool WHOLE = TASKS % THREADS == 0;  // every lane has PER tasks
  unsigned voff[PER];
  float2 v[PER][4];

  __device__ __forceinline__ static int task(int i) {
    return int((threadIdx.x + unsigned(THREADS - FIRST)) % unsigned(THREADS)) + THREADS * i;
  }
  __device__ __forceinline__ static int row_of(int t) { return ROW_CONTIG ? t % ROWS : t / 4; }
  __device__ __forceinline__ static int quad_of(int t) { return ROW_CONTIG ? t / ROWS : t % 4; }

  __device__ __forceinline__ void set_tile(int r0, int nrows, unsigned ld) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int t = task(i), r = r0 + row_of(t), k = 4 * quad_of(t);
      const bool ok = r < nrows && (WHOLE || t < TASKS);
      const unsigned e = !ROW_CONTIG ? unsigned(r) * ld + unsigned(k) : LONG ? unsigned(r) : unsigned(k) * ld + unsigned(r);
      voff[i] = ok ? e * 8u : kOutOfRange;
    }
  }

  // slice starting at reduction index k0 of a tile whose reduction ends at
  // ke, from a matrix of `elems` elements at base. The resource starts at the
  // slice, so that the hardware's range check sees only the lane offsets
  // (ROW_CONTIG: it also ends at the reduction bound). An offset out of range
  // stays so when 3 ld elements are added (ld < 2^25, or LONG, which adds
  // nothing to it and nothing past the reduction).
  __device__ __forceinline__ void load(const float2* base, size_t elems, unsigned ld, int k0, int ke) {
    if (ROW_CONTIG) {
      const __amdgpu_buffer_rsrc_t rs = buffer_resource(base + size_t(k0) * ld, unsigned(ke - k0) * ld * 8u);
#pragma unroll
      for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = 4 * quad_of(task(i)) + j;
          const bool in = voff[i] != kOutOfRange && k < ke - k0;
          v[i][j] = buffer_load_f2(rs, !LONG ? voff[i] + unsigned(j) * ld * 8u
                                       : in  ? voff[i] + unsigned(k) * ld * 8u
                                             : kOutOfRange);
        }
    } else {
      const __amdgpu_buffer_rsrc_t rs = buffer_resource(base + k0, unsigned(elems - size_t(k0)) * 8u);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int k = 4 * quad_of(task(i));
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[i][j] = buffer_load_f2(rs, k + j < ke - k0 ? voff[i] + unsigned(j) * 8u : kOutOfRange);
      }
    }
  }

  // A quad that its pieces lose bits of gets a piece that is NaN, as one with a
  // component too large has already.
  __device__ __forceinline__ void store(uintx4* lds) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int t = task(i);
      if (!WHOLE && t >= TASKS) continue;
      uintx4 q0, q1, q2;
      unsigned lost = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        unsigned a, b, c;
        split3(v[i][j], a, b, c, lost);
        q0[j] = a;
        q1[j] = b;
        q2[j] = c;
      }
      if (static_cast<unsigned short>(lost) != 0) q2[0] = ~0u;
      uintx4* at = lds + quad_at(row_of(t), quad_of(t));
      at[0] = q0;
      at[TASKS] = q1;
      at[2 * TASKS] = q2;
    }
  }
};

constexpr float kMaxFloat = 0x1.fffffep127f;

__device__ __forceinline__ floatx4 mfma(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// One output tile of the logical tile sequence: bin, split, row tile, column
// tile (fastest).
struct MfmaTile {
  int f, split, m0, n0, kb, ke;
};

template <int TM, int TN>
__device__ __forceinline__ MfmaTile mfma_tile(const GemmParams& p, unsigned t, unsigned tiles_m, unsigned tiles_n) {
  MfmaTile c;
  c.n0 = int(t % tiles_n) * TN;
  t /= tiles_n;
  c.m0 = int(t % tiles_m) * TM;
  t /= tiles_m;
  c.split = int(t % unsigned(p.nsplit));
  c.f = unique_bin(int(t / unsigned(p.nsplit)), p.L);
  c.kb = c.split * p.kchunk;
  c.ke = min(p.Kr, c.kb + p.kchunk);
  return c;
}

// LDS of a tile: two buffers of three pieces of both operands' slices.
constexpr size_t mfma_lds_bytes(int TM, int TN) { return size_t(TM + TN) * 4 * 16 * 3 * 2; }

// Persistent matrix-core contraction. MB x NB blocks of 16 x 16 per wave,
// waves in a WM x WN grid: tile (16 WM MB) x (16 WN NB) complex per workgroup.
// The grid (a multiple of 8 workgroups) walks the logical tile sequence in
// rounds; in each round the workgroups of one XCD take consecutive tiles, so
// that tiles sharing operand slices share that XCD's L2. Each workgroup
// streams the reduction slices of all its tiles through one double-buffered
// LDS pipeline: the first slice of its next tile is loaded while the last
// slice of the current one is multiplied.
//
// The complex product is a real one of twice the depth: with rows (ar, ai)
// interleaved, the real part is their product with columns (br, -bi) and the
// imaginary part with (bi, br) (conjugated a: (br, bi) and (bi, -br)), both
// made from the packed (br, bi) in registers. Of the nine products of the
// pieces, the six of order up to 2^-16 are taken; the three left out are
// below 2^-24 of the product, under fp32's own rounding of it (the matrix cores
// take and keep subnormal bf16 and fp32 values). Each slice's
// products are summed in accumulators of their own, the smallest first, and
// added to the tile's once: adding all six straight to the tile's left a
// reduction over 256 tiles at 4.9e-7 relative error against 64 bits, where
// this leaves 3.6e-7 and three fp32 products (Gauss's form, on the fp32
// matrix cores) left 4.1e-7. The matrix cores round toward one side, an error
// of one sign that a sum over many slices or partial results gathers, so every
// other slice is taken with b negated and subtracted: a weight gradient in 43
// partial results of 65 x 56 went from 2.9e-7 relative error to 1.6e-7 (2.0e-7
// on the vector units), that of 128 channels at 56 x 56 from 3.2e-7 to 1.9e-7.
//
// Bound by issue at large sizes. Over the large-kernel layer's three products
// the matrix units are busy 39 - 44 % of the cycles and the other vector
// instructions (the split, the swaps and signs of the packed operand, the
// slices' sums) take another 40 - 44 %; the waves, two per SIMD, wait for their
// turn to issue 35 - 44 % of the time and for data or a barrier 15 - 26 %. The
// clock is at 2.0 - 2.2 GHz. Neither deeper prefetch, nor three workgroups per CU
// on a single buffer, nor the split interleaved with the products moved the
// 1.05 PFLOP/s of bf16 that it runs at. The three products take 0.79, 0.72 and
// 0.73 ms against 0.88, 0.88 and 0.77 on the fp32 matrix cores, those of 128
// channels at 56 x 56 0.25 against 0.29 ms (both in one run).
template <int WM, int WN, int MB, int NB, bool AT, bool AC, bool BT, bool LONG>
__global__ void __launch_bounds__(64 * WM * WN, 2) cgemm_mfma_kernel(GemmParams p, unsigned ntiles) {
  constexpr int TM = 16 * WM * MB, TN = 16 * WN * NB, THREADS = 64 * WM * WN;
  constexpr int QA = TM * 4, QB = TN * 4;  // quads per piece
  extern __shared__ uintx4 lds[];          // [2][3][QA] then [2][3][QB]
  uintx4* const ldsb = lds + 6 * QA;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / WN) * 16 * MB, wn = (wave % WN) * 16 * NB;
  const int lr = lane & 15;  // operand row (A) / column (B) within a 16-block
  const int lk = lane >> 4;  // quad of the slice
  const int fa = quad_at(wm + lr, lk), fb = quad_at(wn + lr, lk);

  const unsigned tiles_m = (p.M + TM - 1) / TM, tiles_n = (p.N + TN - 1) / TN;
  const unsigned nwg = gridDim.x;
  unsigned ct = (blockIdx.x % 8) * (nwg / 8) + blockIdx.x / 8;  // this workgroup's first tile
  if (ct >= ntiles) return;
  MfmaTile cur = mfma_tile<TM, TN>(p, ct, tiles_m, tiles_n);
  int ck = cur.kb;
  // load cursor: one slice ahead of the compute cursor
  unsigned lt = ct;
  MfmaTile nx = cur;
  int lkk = ck;

  Operand<AT, TM, THREADS, 0, LONG> sa;
  Operand<!BT, TN, THREADS, (TM * 4) % THREADS, LONG> sb;
  auto set_tile = [&](const MfmaTile& t) {
    sa.set_tile(t.m0, p.M, unsigned(p.lda));
    sb.set_tile(t.n0, p.N, unsigned(p.ldb));
  };
  auto load_slice = [&](const MfmaTile& t, int k0) {
    sa.load(p.A + size_t(t.f) * p.a_fstride, p.a_fstride, unsigned(p.lda), k0, t.ke);
    sb.load(p.B + size_t(t.f) * p.b_fstride, p.b_fstride, unsigned(p.ldb), k0, t.ke);
  };
  auto advance = [&](unsigned& t, MfmaTile& c, int& k, bool reload) {
    k += kKC;
    if (k >= c.ke) {
      t += nwg;
      if (t < ntiles) {
        c = mfma_tile<TM, TN>(p, t, tiles_m, tiles_n);
        k = c.kb;
        if (reload) set_tile(c);
      }
    }
  };

  set_tile(nx);
  load_slice(nx, lkk);
  sa.store(lds);
  sb.store(ldsb);
  advance(lt, nx, lkk, true);
  __syncthreads();

  floatx4 cr[MB][NB], ci[MB][NB];
  auto zero = [&]() {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        cr[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        ci[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
  };
  zero();

  // The wave's results of a tile in fp32 multiply-adds, with operands straight
  // from memory: where results are infinite or NaN, which they are where the
  // pieces do not hold an operand (see split3). All results of the middle layer
  // (128 channels, 56 x 56) so: 1.3 ms for the forward product, 0.25 without.
  auto again = [&](const MfmaTile& t) {
    zero();
    const float2* A = p.A + size_t(t.f) * p.a_fstride;
    const float2* B = p.B + size_t(t.f) * p.b_fstride;
    unsigned oa[MB][4], ob[NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const unsigned m = unsigned(min(t.m0 + wm + 16 * i + 4 * lk + r, p.M - 1));
        oa[i][r] = AT ? m : m * unsigned(p.lda);
      }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const unsigned n = unsigned(min(t.n0 + wn + 16 * j + lr, p.N - 1));
      ob[j] = BT ? n * unsigned(p.ldb) : n;
    }
#pragma unroll 1
    for (int k = t.kb; k < t.ke; ++k) {
      const unsigned ka = AT ? unsigned(k) * unsigned(p.lda) : unsigned(k);
      const unsigned kb = BT ? unsigned(k) : unsigned(k) * unsigned(p.ldb);
      float2 b[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) b[j] = B[kb + ob[j]];
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float2 a = A[ka + oa[i][r]];
          if (AC) a.y = -a.y;
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            cr[i][j][r] = __builtin_fmaf(-a.y, b[j].y, __builtin_fmaf(a.x, b[j].x, cr[i][j][r]));
            ci[i][j][r] = __builtin_fmaf(a.y, b[j].x, __builtin_fmaf(a.x, b[j].y, ci[i][j][r]));
          }
        }
    }
  };

  int buf = 0;
  for (;;) {
    const bool more = lt < ntiles;
    if (more) load_slice(nx, lkk);
    const uintx4* la = lds + buf * 3 * QA + fa;
    const uintx4* lb = ldsb + buf * 3 * QB + fb;
    // every other slice with b negated, and subtracted
    const bool neg = (unsigned(ck) / kKC) & 1u;
    const unsigned flip = neg ? 0x80008000u : 0u;
    const float sign = neg ? -1.f : 1.f;
    // operand fragments: rows i of A; columns j of the real part, (br, -bi) or
    // with a conjugated (br, bi), and of the imaginary part, (bi, br) or (bi, -br)
    auto rows = [&](int i, bf16x8(&a)[3]) {
#pragma unroll
      for (int q = 0; q < 3; ++q) a[q] = __builtin_bit_cast(bf16x8, la[q * QA + 64 * i]);
    };
    auto columns = [&](int j, bf16x8(&br)[3], bf16x8(&bi)[3]) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const uintx4 b = lb[q * QB + 64 * j];
        uintx4 re, im;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned swapped = __builtin_amdgcn_alignbit(b[e], b[e], 16);
          re[e] = b[e] ^ (flip ^ (AC ? 0u : 0x80000000u));
          im[e] = swapped ^ (flip ^ (AC ? 0x80000000u : 0u));
        }
        br[q] = __builtin_bit_cast(bf16x8, re);
        bi[q] = __builtin_bit_cast(bf16x8, im);
      }
    };
    // half way through the products, the slice loaded at their start goes to the
    // buffer that the previous barrier released
    auto next_slice = [&]() {
      if (!more) return;
      sa.store(lds + (buf ^ 1) * 3 * QA);
      sb.store(ldsb + (buf ^ 1) * 3 * QB);
    };
    constexpr bool A_STAYS = 20 * MB + 24 < 32 * NB + 12;  // registers of either order
    if constexpr (A_STAYS) {
      bf16x8 a[MB][3];
#pragma unroll
      for (int i = 0; i < MB; ++i) rows(i, a[i]);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        if (j == (NB + 1) / 2) next_slice();
        bf16x8 br[3], bi[3];
        columns(j, br, bi);
        floatx4 tr[MB], ti[MB];
#pragma unroll
        for (int i = 0; i < MB; ++i) tr[i] = ti[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int order = 2; order >= 0; --order)
#pragma unroll
          for (int pa = order; pa >= 0; --pa)
#pragma unroll
            for (int i = 0; i < MB; ++i) {
              tr[i] = mfma(a[i][pa], br[order - pa], tr[i]);
              ti[i] = mfma(a[i][pa], bi[order - pa], ti[i]);
            }
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          cr[i][j] += sign * tr[i];
          ci[i][j] += sign * ti[i];
        }
      }
      if (NB == 1) next_slice();
    } else {
      bf16x8 br[NB][3], bi[NB][3];
#pragma unroll
      for (int j = 0; j < NB; ++j) columns(j, br[j], bi[j]);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (i == (MB + 1) / 2) next_slice();
        bf16x8 a[3];
        rows(i, a);
        floatx4 tr[NB], ti[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) tr[j] = ti[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int order = 2; order >= 0; --order)
#pragma unroll
          for (int pa = order; pa >= 0; --pa)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              tr[j] = mfma(a[pa], br[j][order - pa], tr[j]);
              ti[j] = mfma(a[pa], bi[j][order - pa], ti[j]);
            }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          cr[i][j] += sign * tr[j];
          ci[i][j] += sign * ti[j];
        }
      }
      if (MB == 1) next_slice();
    }
    __builtin_amdgcn_s_setprio(0);
    if (ck + kKC >= cur.ke) {
      // the largest result, or NaN if there is one (maximum, not max)
      float most[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            most[r] = __builtin_elementwise_maximum(
                most[r], __builtin_elementwise_maximum(__builtin_fabsf(cr[i][j][r]), __builtin_fabsf(ci[i][j][r])));
      const float all = __builtin_elementwise_maximum(__builtin_elementwise_maximum(most[0], most[1]),
                                                      __builtin_elementwise_maximum(most[2], most[3]));
      if (__builtin_expect(__any(!(all <= kMaxFloat)), 0)) again(cur);
      // 16 x 16 result block: lane holds rows 4*(lane/16) + r, r < 4, of column
      // lane % 16; each bin's matrix is under 2^28 elements (32-bit offsets)
      float2* Cm = p.C + size_t(cur.f) * p.c_fstride + size_t(cur.split) * p.c_sstride;
      const unsigned ldc = unsigned(p.ldc);
      const int mb = cur.m0 + wm + 4 * lk, nb = cur.n0 + wn + lr;
      if (cur.m0 + TM <= p.M && cur.n0 + TN <= p.N) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float2* row = Cm + unsigned(mb + 16 * i + r) * ldc + unsigned(nb);
#pragma unroll
            for (int j = 0; j < NB; ++j) row[16 * j] = make_float2(cr[i][j][r], ci[i][j][r]);
          }
      } else {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = mb + 16 * i + r;
            float2* row = Cm + unsigned(m) * ldc + unsigned(nb);
#pragma unroll
            for (int j = 0; j < NB; ++j)
              if (m < p.M && nb + 16 * j < p.N) row[16 * j] = make_float2(cr[i][j][r], ci[i][j][r]);
          }
      }
      zero();
    }
    __syncthreads();
    if (!more) break;
    buf ^= 1;
    advance(ct, cur, ck, false);
    advance(lt, nx, lkk, true);
  }
}

template <int WM, int WN, int MB, int NB, bool AT, bool AC, bool BT, bool LONG = false>
hipError_t launch_mfma_shape(const GemmParams& p, hipStream_t s) {
  constexpr int TM = 16 * WM * MB, TN = 16 * WN * NB, threads = 64 * WM * WN;
  constexpr size_t lds = mfma_lds_bytes(TM, TN);
  const unsigned long long tiles = (unsigned long long)((p.M + TM - 1) / TM) * ((p.N + TN - 1) / TN) *
                                   unsigned(p.nsplit) * unsigned(p.F);
  if (tiles == 0) return hipSuccess;
  if (tiles > 0xffffffffull) return hipErrorInvalidValue;
  auto kern = cgemm_mfma_kernel<WM, WN, MB, NB, AT, AC, BT, LONG>;
  hipError_t e = lds > 65536 ? tile::allow_lds(kern, lds) : hipSuccess;
  if (e != hipSuccess) return e;
  // resident workgroups of this instantiation, queried once per device
  static std::atomic<int> resident[64];
  int dev = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  int groups = resident[dev].load(std::memory_order_relaxed);
  if (groups == 0) {
    int cus = 0, per_cu = 0;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, lds)) != hipSuccess) return e;
    groups = (per_cu < 1 ? 1 : per_cu) * (cus < 1 ? 1 : cus);
    resident[dev].store(groups, std::memory_order_relaxed);
  }
  unsigned long long nwg = (unsigned long long)(groups) < tiles ? groups : tiles;
  nwg = (nwg + 7) / 8 * 8;  // whole rounds over the 8 XCDs
  hipLaunchKernelGGL(kern, dim3(unsigned(nwg)), dim3(threads), lds, s, p, unsigned(tiles));
  return hipGetLastError();
}

// Row-contiguous operands with rows under 2^25 elements: the offsets of 16
// reduction indices fit 32 bits.
bool rows_short(const GemmParams& p) {
  const long lim = 1l << 25;
  return (!p.a_trans || p.lda < lim) && (p.b_trans || p.ldb < lim);
}

// The tile shape with the least estimated time.
template <bool AT, bool AC, bool BT>
hipError_t launch_mfma(const GemmParams& p, hipStream_t s) {
  if (!rows_short(p)) return launch_mfma_shape<1, 4, 1, 2, AT, AC, BT, true>(p, s);
  using Launch = hipError_t (*)(const GemmParams&, hipStream_t);
  static constexpr Launch kLaunch[] = {
      launch_mfma_shape<1, 4, 1, 1, AT, AC, BT>, launch_mfma_shape<1, 4, 1, 2, AT, AC, BT>,
      launch_mfma_shape<4, 1, 1, 1, AT, AC, BT>, launch_mfma_shape<2, 2, 1, 1, AT, AC, BT>,
      launch_mfma_shape<2, 2, 1, 2, AT, AC, BT>, launch_mfma_shape<2, 2, 2, 1, AT, AC, BT>,
      launch_mfma_shape<2, 2, 2, 2, AT, AC, BT>, launch_mfma_shape<2, 2, 3, 2, AT, AC, BT>,
      launch_mfma_shape<2, 2, 2, 3, AT, AC, BT>, launch_mfma_shape<2, 2, 4, 2, AT, AC, BT>,
      launch_mfma_shape<2, 2, 3, 3, AT, AC, BT>, launch_mfma_shape<4, 2, 2, 3, AT, AC, BT>,
      launch_mfma_shape<2, 4, 3, 2, AT, AC, BT>, launch_mfma_shape<2, 4, 4, 2, AT, AC, BT>,
  };  // in the order of kMfmaTiles
  static_assert(sizeof kLaunch / sizeof kLaunch[0] == sizeof kMfmaTiles / sizeof kMfmaTiles[0], "one per shape");
  return kLaunch[mfma_tile_choice(p.M, p.N, p.Kr, p.kchunk, p.nsplit, p.F)](p, s);
}

template <int TM, int TN, class Kern>
hipError_t launch(Kern kern, const GemmParams& p, hipStream_t s) {
  const unsigned tiles = unsigned(((p.M + TM - 1) / TM) * ((p.N + TN - 1) / TN));
  hipLaunchKernelGGL(kern, dim3(tiles, unsigned(p.nsplit), unsigned(p.F)), dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

// The matrix-core path reads each bin's operands and writes its result through
// 32-bit byte offsets.
bool mfma_addressable(const GemmParams& p) {
  const size_t lim = size_t(1) << 28;
  return p.a_fstride < lim && p.b_fstride < lim && p.c_fstride < lim && size_t(p.M) * size_t(p.ldc) < lim;
}

}  // namespace

hipError_t launch_cgemm_valu(const GemmParams& p, hipStream_t s) {
  if (p.kchunk % kKC != 0 && p.nsplit > 1) return hipErrorInvalidValue;
  // the three operand orientations of the layer's passes, and the plain
  // product that composes two layers' kernel spectra
  if (p.a_trans && !p.a_conj && !p.b_trans && !p.b_conj)
    return launch<kVM, kVN>(cgemm_valu_kernel<true, false, false, false>, p, s);
  if (!p.a_trans && p.a_conj && !p.b_trans && !p.b_conj)
    return launch<kVM, kVN>(cgemm_valu_kernel<false, true, false, false>, p, s);
  if (!p.a_trans && p.a_conj && p.b_trans && !p.b_conj)
    return launch<kVM, kVN>(cgemm_valu_kernel<false, true, true, false>, p, s);
  if (!p.a_trans && !p.a_conj && !p.b_trans && !p.b_conj)  // kernel spectra of two stacked layers
    return launch<kVM, kVN>(cgemm_valu_kernel<false, false, false, false>, p, s);
  return hipErrorInvalidValue;
}

hipError_t launch_cgemm_mfma(const GemmParams& p, hipStream_t s) {
  if (p.kchunk % kKC != 0 && p.nsplit > 1) return hipErrorInvalidValue;
  if (!mfma_addressable(p)) return hipErrorInvalidValue;
  if (p.a_trans && !p.a_conj && !p.b_trans && !p.b_conj) return launch_mfma<true, false, false>(p, s);
  if (!p.a_trans && p.a_conj && !p.b_trans && !p.b_conj) return launch_mfma<false, true, false>(p, s);
  if (!p.a_trans && p.a_conj && p.b_trans && !p.b_conj) return launch_mfma<false, true, true>(p, s);
  if (!p.a_trans && !p.a_conj && !p.b_trans && !p.b_conj) return launch_mfma<false, false, false>(p, s);
  return hipErrorInvalidValue;
}

bool mfma_fits(const GemmParams& p) { return mfma_addressable(p) && rows_short(p); }

}  // namespace oaa
