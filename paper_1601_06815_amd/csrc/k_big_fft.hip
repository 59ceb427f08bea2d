// Transforms of side L = 64 (arXiv:1601.06815, Section 2: block division, zero
// padding, the per-block transforms and the overlap-add of the block results;
// Section 3.3 for the transform sides of large kernels), as used for large
// blocks (b up to L - n + 1) and large kernels, in launches of many tiles; and
// the launchers of both large sides, which give L = 128 and launches of few
// tiles to k_wide_fft.hip.
//
// A workgroup keeps the intermediate of TQ tiles in LDS (17 KB per tile, so
// one workgroup of up to nine tiles per CU) and walks over groups of TQ
// consecutive tiles of one channel:
//  * forward: pass 1 transforms the column pairs (s, s + L/2) of every window
//    along its rows, lanes over consecutive columns so that the loads of a
//    row are coalesced, and keeps rows u <= L/2 of the two real columns'
//    spectra (rows past L/2 are their conjugates); pass 2 transforms each of
//    those rows along the columns and writes bins (u, v) and (L - u, v) of
//    the half spectrum with lanes over the group's tiles, so that a store
//    instruction writes runs of TQ consecutive tiles of a bin. Consecutive
//    groups run on one XCD at about the same time, so the runs that
//    neighbouring groups write into a bin meet in that XCD's L2;
//  * inverse: pass 1 inverts the columns v <= L/2 (loads in runs of TQ
//    tiles), pass 2 inverts row pairs to real rows, pass 3 writes the kept
//    part of each tile (crop) or the overlap-added plane. Teams of workgroups
//    of one XCD take neighbouring groups together, each team walking a
//    contiguous range, so that the 128-byte lines that those groups' runs
//    share come from HBM once.
// A lane holds a whole 64-point sequence, and the two halves of the workgroup
// alternate between transforming a group and loading the next into their
// registers (big_rfft2_lane_kernel, big_irfft2_lane_kernel).
#include <algorithm>
#include <type_traits>

#include "fft_core.hpp"
#include "oaa_internal.hpp"
#include "tile_common.hpp"

namespace oaa {

namespace {

using namespace tile;

constexpr size_t kBigLds = 160 * 1024;  // LDS of one CU

// Tiles per group (overridable at build time for tuning sweeps).
#ifndef OAA_BIG_TQ
#define OAA_BIG_TQ 8
#endif

struct Big {
  static constexpr int L = 64, H2 = L / 2, V = L / 2 + 1;
  // forward LDS row stride (complex): columns [0, L/2) then, one slot on,
  // columns [L/2, L)
  static constexpr int RS = L + 2;
  // inverse LDS row stride (complex): L/2 slots, slot 0 holding the real
  // columns 0 and L/2 as (re, im), plus one slot of padding
  static constexpr int RI = H2 + 1;
  static constexpr int TQ_MAX = 9;    // tiles per group (LDS)
  static constexpr int SIDE_MAX = 3;  // blocks per side of a one-group plane
};

// LDS per tile (complex elements): the 32 x 66
// (forward) or 64 x 33 (inverse) slots, padded to 3 mod 32, so that tile
// bases fall 6 four-byte banks apart. A wave's lanes over (tile, LDS row) in
// the forward's second pass, and over (tile, column) or (tile, row pair) in
// the inverse's passes, then spread over the banks; at the odd stride 1 mod
// 32, neighbouring tiles fell 2 banks apart, on the banks of the next row or
// column (measured at the large-kernel layer: forward inverse 0.621 ->
// 0.615 ms).
__host__ __device__ constexpr int lane_tile_stride() {
  constexpr int n = 64 * Big::RI;
  static_assert(n == 32 * Big::RS, "both directions hold 2112 complex per tile");
  return n + ((3 - n % 32) + 32) % 32;
}

// first group of this workgroup; groups advance by gridDim.x (a multiple of
// 8), and the workgroups of one XCD take consecutive groups
__device__ __forceinline__ long first_group() {
  const unsigned nwg = gridDim.x;
  return long(blockIdx.x % 8) * (nwg / 8) + blockIdx.x / 8;
}

// The groups a workgroup takes: g, g + step, ... below end. The forward
// transform walks interleaved: consecutive groups on the workgroups of one
// XCD at about the same time.
struct GroupWalk {
  long g, end, step;
};
__device__ __forceinline__ GroupWalk group_walk(long ngroups) { return {first_group(), ngroups, long(gridDim.x)}; }

// Teams of S workgroups of one XCD (consecutive first_group numbers; nwg is
// a multiple of 8 S, else S is 1) take S consecutive groups at a time, and
// each team walks a contiguous range. The runs of S neighbouring groups in a
// bin share 128-byte lines, which the first of them to read one brings into
// the XCD's L2 for the others, read at about the same time. A line shared by
// groups a workgroup takes one after the other is gone from L2 by the next
// group (a workgroup's group reads 2050 bins), so a contiguous walk with S = 1
// reads each such line again. A team of a whole XCD on one channel at a time
// (S = 32, like the interleaved walk) crowds all XCDs onto a few channels'
// bins and was slower. Measured at the large-kernel layer (groups of one
// nine-tile plane in the forward overlap-add, of 8 tiles = 64 bytes in the
// crops): forward inverse 0.675 / 0.625 / 0.622 / 0.694 ms at S = 1, 4, 8,
// 16; the crops 0.224 -> 0.217 and 0.151 -> 0.142 ms at S = 2, where a pair
// of groups covers one line.
__device__ __forceinline__ GroupWalk group_walk_team(long ngroups, int S0) {
  const long w = first_group(), nwg = gridDim.x;
  const long S = nwg % (8 * S0) == 0 ? S0 : 1;
  const long R = (ngroups + nwg - 1) / nwg, team = w / S, s = w % S;
  return {team * R * S + s, min(ngroups, (team + 1) * R * S), S};
}

// ---------------------------------------------------------------------------
// forward: windows of planes -> half spectra, a whole 64-point sequence per
// lane.
//
// Pass 1: z = x[., j] + i x[., j + L/2] along the rows; the real columns'
// spectra are C_j[u] = (Z[u] + conj Z[-u]) / 2, C_{j+L/2}[u] =
// (Z[u] - conj Z[-u]) / (2i), Hermitian in u, so rows u <= L/2 suffice; rows
// 0 and L/2 are real and share LDS row 0 as (re, im). Pass 2: rows u in
// [1, L/2) along the columns give bins (u, v), v <= L/2, and (L - u, v) =
// conj X[u][L - v], 0 < v < L/2 (the other bins of rows past L/2 are
// conjugates that nothing reads); the packed row gives rows 0 and L/2 by the
// same separation as pass 1. Against a transform split over a lane pair, with
// its first stage across the pair, one lane takes about 0.7 of the vector
// instructions. The 32 tasks per tile and pass of a group of eight tiles fill
// four waves, half the workgroup, and the halves alternate: while one
// transforms group i, the other loads the windows of group i + 1 into its
// registers, so the loads have a whole group's passes to arrive. A half's
// pass 2 works in the registers that held its windows.
//
// A wave holds the column pairs of two tiles, possibly of two images, and a
// buffer resource must be the same for the whole wave: the window rows come
// through one resource per group, over the planes of channel ch of the
// group's images. WIDE: spans of the planes or spectra past 32-bit offsets,
// through 64-bit addresses.
template <bool WIDE>
__global__ void __launch_bounds__(512) big_rfft2_lane_kernel(BigFwdParams p) {
  constexpr int L = 64, H2 = L / 2, V = L / 2 + 1, RS = Big::RS;
  extern __shared__ float smem[];
  float2* lds = reinterpret_cast<float2*>(smem);
  const int TSZ = lane_tile_stride();
  const int tid = threadIdx.x, TQ = p.TQ;
  const int half = tid >> 8, ht = tid & 255;  // half of the workgroup (four waves), thread in it
  const int P = p.T * p.T, tpc = p.n_img * P;
  const size_t bs = p.bs;
  const long ngroups = long(p.n_ch) * p.ngrp;
  const size_t HH = size_t(p.H) * p.H, istride = size_t(p.n_ch) * HH;  // floats per plane, per image
  // this thread's tasks: pass 1 tile q1, column pair j (lanes over consecutive
  // columns: coalesced window rows); pass 2 tile q2, LDS row u (lanes over
  // the tiles: runs of consecutive tiles of a bin)
  const int q1 = ht / H2, j = ht % H2, q2 = ht % TQ, u = ht / TQ;
  float zr[L], zi[L];

  // the windows of group g: columns j and j + L/2 of tile q1 as
  // z = x[., j] + i x[., j + L/2]
  auto fetch = [&](long g) {
    const int ch = int(g / p.ngrp), t0 = int(g % p.ngrp) * TQ;
    const int nq = min(TQ, tpc - t0);
    if (q1 >= nq) return;
    const int img0 = t0 / P, img1 = (t0 + nq - 1) / P;
    const float* base = p.src + (size_t(img0) * p.n_ch + ch) * HH;
    const __amdgpu_buffer_rsrc_t rs =
        buffer_resource(base, WIDE ? 0u : unsigned((size_t(img1 - img0) * istride + HH) * 4));
    const int t = t0 + q1, img = t / P, pp = t - img * P;
    const int pr = pp / p.T, qc = pp - pr * p.T;
    const int gr0 = pr * p.pitch - p.off;
    const int ca = qc * p.pitch - p.off + j, cb = ca + H2;
    const bool oka = j < p.S && unsigned(ca) < unsigned(p.H);
    const bool okb = j + H2 < p.S && unsigned(cb) < unsigned(p.H);
    const unsigned pb = unsigned(size_t(img - img0) * istride);  // this tile's plane in rs (elements)
    const float* plane = p.src + (size_t(img) * p.n_ch + ch) * HH;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int gr = gr0 + i;
      const bool okr = i < p.S && unsigned(gr) < unsigned(p.H);
      if (WIDE) {
        zr[i] = okr && oka ? plane[size_t(gr) * p.H + ca] : 0.f;
        zi[i] = okr && okb ? plane[size_t(gr) * p.H + cb] : 0.f;
      } else {
        zr[i] = buffer_load_f1(rs, okr && oka ? (pb + unsigned(gr * p.H + ca)) * 4u : kOutOfRange);
        zi[i] = buffer_load_f1(rs, okr && okb ? (pb + unsigned(gr * p.H + cb)) * 4u : kOutOfRange);
      }
    }
  };
  // pass 1 on the fetched windows: the real columns' spectra
  // C_j[u] = (Z[u] + conj Z[L - u]) / 2, C_{j+L/2}[u] = (Z[u] - conj Z[L - u]) / (2i),
  // rows u <= L/2; rows 0 and L/2 (real) share LDS row 0 as (re, im)
  auto columns = [&]() {
    fft_dif<L, -1, false>(zr, zi);  // Z[k] at position bitrev(k)
    float2* bq = lds + (q1 * TSZ + j);
#pragma unroll
    for (int v = 1; v < H2; ++v) {
      const float a = zr[bitrev(v, L)], b = zi[bitrev(v, L)];
      const float c = zr[bitrev(L - v, L)], d = zi[bitrev(L - v, L)];
      bq[v * RS] = make_float2(0.5f * (a + c), 0.5f * (b - d));
      bq[v * RS + H2 + 1] = make_float2(0.5f * (b + d), 0.5f * (c - a));
    }
    bq[0] = make_float2(zr[0], zr[bitrev(H2, L)]);
    bq[H2 + 1] = make_float2(zi[0], zi[bitrev(H2, L)]);
  };
  // pass 2: LDS row u of tile q2 along the columns; bins (u, v), v <= L/2,
  // and (L - u, v) = conj X[u][L - v], 0 < v < L/2; the packed row 0 gives
  // rows 0 and L/2 by the separation of pass 1
  auto row = [&](int ch, int t0) {
    const float2* zrow = lds + (q2 * TSZ + u * RS);
#pragma unroll
    for (int c = 0; c < H2; ++c) {
      const float2 a = zrow[c], b = zrow[H2 + 1 + c];
      zr[c] = a.x;
      zi[c] = a.y;
      zr[H2 + c] = b.x;
      zi[H2 + c] = b.y;
    }
    fft_dif<L, -1, false>(zr, zi);  // Y[v] at position bitrev(v)
    const int t = t0 + q2;
    const size_t tb = size_t(ch) * p.cs + size_t(t / p.run) * p.rs + size_t(t % p.run);
    auto put = [&](int r, int v, float2 val) {
      if (!WIDE) {
        store_at(p.dst, unsigned((size_t(r) * V * bs + tb) * 8u) + unsigned(v) * unsigned(bs * 8u), val);
      } else {
        p.dst[(size_t(r) * V + v) * bs + tb] = val;
      }
    };
    if (u > 0) {
#pragma unroll
      for (int v = 0; v <= H2; ++v) put(u, v, make_float2(zr[bitrev(v, L)], zi[bitrev(v, L)]));
#pragma unroll
      for (int v = 1; v < H2; ++v) put(L - u, v, make_float2(zr[bitrev(L - v, L)], -zi[bitrev(L - v, L)]));
    } else {
#pragma unroll
      for (int v = 0; v <= H2; ++v) {
        const float a = zr[bitrev(v, L)], b = zi[bitrev(v, L)];
        const float c = zr[bitrev((L - v) % L, L)], d = zi[bitrev((L - v) % L, L)];
        put(0, v, make_float2(0.5f * (a + c), 0.5f * (b - d)));
        put(H2, v, make_float2(0.5f * (b + d), 0.5f * (c - a)));
      }
    }
  };

  const GroupWalk wk = group_walk(ngroups);
  if (half == 0 && wk.g < wk.end) fetch(wk.g);
  int turn = 0;  // the half whose windows are in registers for this group
  for (long g = wk.g; g < wk.end; g += wk.step, turn ^= 1) {
    const int ch = int(g / p.ngrp), t0 = int(g % p.ngrp) * TQ;
    const int nq = min(TQ, tpc - t0);
    const bool mine = half == turn;
    if (mine) {
      if (q1 < nq) columns();
    } else if (g + wk.step < wk.end) {
      fetch(g + wk.step);
    }
    __syncthreads();
    if (mine && q2 < nq && u < H2) row(ch, t0);
    __syncthreads();
  }
}

// Output of a group that is one whole plane, from its real tiles in LDS (tile
// q at float offset 2 q TSZ, row r of a tile at 2 r RI): output pixel (i, j)
// is framed pixel (i + off, j + off), the sum of at most two tiles per side,
// added in a fixed order. A wave per output row, lanes over the columns. Each
// lane's column offsets in the (at most two) tiles covering its columns, with
// 0/1 weights, are taken once per plane, so that the reads of a row need no
// per-lane branch; the tile rows covering a row are the same for the whole
// wave. Rows and columns are at their inverse index r, kept index
// (r + rot) mod L, and hold L^2 times the values.
__device__ __forceinline__ void overlap_plane_out(const BigInvParams& p, const float* ldf, int TSZ, int ch, int t0,
                                                  int wave, int lane, int nwave) {
  constexpr int RI = Big::RI, L = 64;
  const int H = p.H, KR = p.KR, P = p.T * p.T;
  // stored index of kept index k
  auto at = [&](int k) { return (k - p.rot) & (L - 1); };
  const float wt = 1.0f / float(L * L);
  const int img = t0 / P, T = p.T, b = p.pitch;
  float* out = p.dst + (size_t(img) * p.n_ch + ch) * H * H;
  const SmallDiv div_b(b);
  constexpr int MCH = (L * Big::SIDE_MAX + 63) / 64;  // H < T b <= L T
  int o0[MCH], o1[MCH];
  float m0[MCH], m1[MCH];
  int ln = lane;  // opaque: the offsets are not kept across the group loop
  asm volatile("" : "+v"(ln));
#pragma unroll
  for (int k = 0; k < MCH; ++k) {
    const int jx = ln + 64 * k, c = jx + p.off, Q1 = div_b(c), ca1 = c - Q1 * b;
    const bool in = jx < H;
    const bool v1 = in && Q1 < T, v0 = in && Q1 >= 1 && Q1 - 1 < T && ca1 + b < KR;
    o0[k] = v0 ? (Q1 - 1) * TSZ * 2 + at(ca1 + b) : 0;
    o1[k] = v1 ? Q1 * TSZ * 2 + at(ca1) : 0;
    m0[k] = v0 ? 1.f : 0.f;
    m1[k] = v1 ? 1.f : 0.f;
  }
  const int nch = (H + 63) / 64;
  for (int i = wave; i < H; i += nwave) {
    const int a = i + p.off, P1 = div_b(a), ra1 = a - P1 * b;
    // tile rows covering framed row a: P1 (row ra1) and P1 - 1 (row ra1 + b)
    const bool r1 = P1 < T, r0 = P1 >= 1 && P1 - 1 < T && ra1 + b < KR;
    const float* l1 = ldf + (r1 ? 2 * (P1 * T * TSZ + at(ra1) * RI) : 0);
    const float* l0 = ldf + (r0 ? 2 * ((P1 - 1) * T * TSZ + at(ra1 + b) * RI) : 0);
    const float w0 = r0 ? wt : 0.f, w1 = r1 ? wt : 0.f;
    float* orow = out + size_t(i) * H;
    float acc[MCH];
#pragma unroll
    for (int k = 0; k < MCH; ++k) {
      if (k >= nch) break;
      const float t0v = __builtin_fmaf(m0[k], l0[o0[k]], m1[k] * l0[o1[k]]);
      const float t1v = __builtin_fmaf(m0[k], l1[o0[k]], m1[k] * l1[o1[k]]);
      acc[k] = __builtin_fmaf(w0, t0v, w1 * t1v);
    }
#pragma unroll
    for (int k = 0; k < MCH; ++k) {
      if (k >= nch) break;
      const int jx = lane + 64 * k;
      if (jx < H) orow[jx] = acc[k];
    }
  }
}

// ---------------------------------------------------------------------------
// inverse: half spectra -> kept part of every tile (crop), or the plane the
// tiles overlap-add to, a whole 64-point sequence per lane.
//
// Pass 1 inverts column w of every tile, w < L/2; column 0 carries the real
// columns 0 and L/2 together as h0[u] + i h1[u] (rows past L/2 rebuilt as the
// conjugates of rows L - u, which are not stored), so its inverse holds both
// real columns. Pass 2 inverts pairs of rows to real rows, written over their
// own storage. The 32 tasks per tile and pass of a group of eight tiles
// fill four waves, half the workgroup, and the halves alternate: while one
// transforms group i, the other loads the columns of group i + 1 into its
// registers, which then have passes 2 and 3 of group i to arrive. A nine-tile
// plane has 32 tasks per pass past the half's 256; the loading half runs
// them (loading their columns itself) before it loads the next group.
// Pass 3, the output, takes all eight waves.
//
// Rows and columns stay in LDS at their inverse index r (kept index
// (r + rot) mod L), in tiles of L x (L/2 + 1) slots, so that every LDS
// address is a compile-time offset from the task's base; passes 1 and 2
// write every row and column (skipping the ones nothing reads, under
// conditions that are uniform, makes the compiler keep more of the
// transform's values live across the stores, and spill), pass 2 runs on the
// row pairs that hold kept rows only, and the output pass applies the
// rotation and the 1/L^2 scale. MODE: the kernel's pass 3 (0 crop, 1
// overlap-add of one-group planes), fixed per instance so that each carries
// only the registers of its own output code; SPLIT: more
// than one partial spectrum to sum (the weight gradient's split), loaded in
// batches of 16 rows so that the partial sums and the loads in flight fit
// the registers.
template <bool O32, int MODE, bool SPLIT>
__global__ void __launch_bounds__(512) big_irfft2_lane_kernel(BigInvParams p) {
  constexpr int L = 64, H2 = L / 2, V = L / 2 + 1, RI = Big::RI, HALF = 256;
  extern __shared__ float smem[];
  float2* lds = reinterpret_cast<float2*>(smem);
  const float* ldf = smem;
  const int KR = p.KR, rot = p.rot, TQ = p.TQ;
  const int TSZ = lane_tile_stride();
  const int tid = threadIdx.x;
  const int half = tid >> 8, ht = tid & (HALF - 1);  // half of the workgroup (four waves), thread in it
  const int P = p.T * p.T, tpc = p.n_img * P;
  const size_t fstride = size_t(p.n_ch) * tpc;
  const long ngroups = long(p.n_ch) * p.ngrp;
  // the stored rows (k - rot) mod L of kept rows k < KR are a cyclic run
  // from s0; the row pairs w0, w0 + 1, ... (mod L/2) cover it
  const int s0 = (L - rot) & (L - 1), w0 = s0 >> 1, npair = min(H2, ((s0 & 1) + KR + 1) >> 1);
  const int ntask1 = H2 * TQ, ntask2 = npair * TQ;  // tasks of passes 1 and 2 (tile fastest)
  using off_t = typename std::conditional<O32, unsigned, size_t>::type;
  auto at = [&](const float2* base, off_t e) { return O32 ? load_at(base, unsigned(e) * 8u) : base[e]; };
  float re[L], im[L];  // a lane's sequence: loaded columns, then the pass's working values

  // column w of tile q into re/im (summed over the partial spectra); column
  // 0 carries the real columns 0 and L/2 together as h0[u] + i h1[u], rows
  // past L/2 rebuilt as the conjugates of rows L - u (not stored)
  auto fetch = [&](int ch, int t0, int q, int w) __attribute__((always_inline)) {
    const size_t tb = size_t(ch) * tpc + t0 + q;
    const off_t row = off_t(size_t(V) * fstride);
    // rows [u0, u0 + NU) of one partial: assigned (first) or added
    auto gather = [&](const float2* base, int u0c, auto nu, auto first) __attribute__((always_inline)) {
      constexpr int NU = decltype(nu)::value;
      constexpr bool FIRST = decltype(first)::value;
      const int u0 = u0c;
      if (w > 0) {
        off_t e = off_t((size_t(u0) * V + w) * fstride + tb);
        if (O32) asm volatile("" : "+v"(e));
#pragma unroll
        for (int i = 0; i < NU; ++i) {
          const float2 z = at(base, e);
          e += row;
          re[u0 + i] = FIRST ? z.x : re[u0 + i] + z.x;
          im[u0 + i] = FIRST ? z.y : im[u0 + i] + z.y;
        }
      } else {
        // rows u <= L/2 of columns 0 and L/2 give rows u and L - u
        off_t e = off_t(size_t(u0) * V * fstride + tb);
        if (O32) asm volatile("" : "+v"(e));
        const off_t hoff = off_t(size_t(H2) * fstride);
#pragma unroll
        for (int i = 0; i < NU; ++i) {
          const int u = u0 + i;
          if (u > H2) break;
          const float2 b0 = at(base, e), b1 = at(base, e + hoff);
          e += row;
          re[u] = FIRST ? b0.x - b1.y : re[u] + (b0.x - b1.y);
          im[u] = FIRST ? b0.y + b1.x : im[u] + (b0.y + b1.x);
          if (u > 0 && u < H2) {
            re[L - u] = FIRST ? b0.x + b1.y : re[L - u] + (b0.x + b1.y);
            im[L - u] = FIRST ? b1.x - b0.y : im[L - u] + (b1.x - b0.y);
          }
        }
      }
    };
    if constexpr (!SPLIT) {
      gather(p.src, 0, std::integral_constant<int, L>{}, std::true_type{});
    } else {
      // column 0 reads rows [0, L/2] only, which the first three batches
      // cover (the fourth then reads nothing)
#pragma unroll
      for (int u0 = 0; u0 < L; u0 += 16) {
        gather(p.src, u0, std::integral_constant<int, 16>{}, std::true_type{});
        for (int sp = 1; sp < p.nsplit; ++sp)
          gather(p.src + size_t(sp) * p.split_stride, u0, std::integral_constant<int, 16>{}, std::false_type{});
        asm volatile("" ::: "memory");
      }
    }
  };
  // pass 1 on the fetched column w of tile q
  auto column = [&](int q, int w) __attribute__((always_inline)) {
    fft_dif<L, +1, false>(re, im);  // row r at position bitrev(r)
    float2* bq = lds + (q * TSZ + w);
#pragma unroll
    for (int r = 0; r < L; ++r) bq[r * RI] = make_float2(re[bitrev(r, L)], im[bitrev(r, L)]);
  };
  // pass 2: rows 2w, 2w + 1 to L^2 times their real rows, written over their
  // own storage (slot 0 of a row holds its bins 0 and L/2 as (re, im))
  auto rows = [&](int q, int w) __attribute__((always_inline)) {
    float2* za = lds + (q * TSZ + 2 * w * RI);
    {
      const float2 a0 = za[0], b0 = za[RI];
      re[0] = a0.x;
      im[0] = b0.x;
      re[H2] = a0.y;
      im[H2] = b0.y;
    }
#pragma unroll
    for (int v = 1; v < H2; ++v) {
      const float2 a = za[v], bb = za[RI + v];
      re[v] = a.x - bb.y;
      im[v] = a.y + bb.x;
      re[L - v] = a.x + bb.y;
      im[L - v] = bb.x - a.y;
    }
    fft_dif<L, +1, false>(re, im);  // L^2 row0[s] in re, L^2 row1[s] in im, at position bitrev(s)
    float* d0 = reinterpret_cast<float*>(za);
#pragma unroll
    for (int s = 0; s < L; ++s) {
      d0[s] = re[bitrev(s, L)];
      d0[2 * RI + s] = im[bitrev(s, L)];
    }
  };
  // pass 3, MODE 0: the kept KR x KR of every tile, scaled, to its block; a
  // wave per tile (decoded once, wave-uniform), lanes over the block in row order
  auto crop = [&](int ch, int t0, int nq, int wave, int lane, int nwave, auto rotated) {
    constexpr bool ROT = decltype(rotated)::value;
    const float scale = 1.0f / float(L * L);
    const SmallDiv div_k(KR);
    for (int qq = wave; qq < nq; qq += nwave) {
      const float* lt = ldf + 2 * qq * TSZ;
      const int t = t0 + qq, img = t / P, pp = t - img * P;
      const int pr = pp / p.T, qc = pp - pr * p.T;
      const int nrow = min(KR, p.H - pr * p.pitch), ncol = min(KR, p.H - qc * p.pitch);
      float* ob = p.dst + ((size_t(img) * p.n_ch + ch) * p.H + pr * p.pitch) * p.H + qc * p.pitch;
      for (int e = lane; e < KR * nrow; e += 64) {
        const int rr = div_k(e), cc = e - rr * KR;
        const int sr = ROT ? (rr - rot) & (L - 1) : rr, sc = ROT ? (cc - rot) & (L - 1) : cc;
        if (cc < ncol) ob[rr * p.H + cc] = lt[2 * sr * RI + sc] * scale;
      }
    }
  };

  const GroupWalk wk = group_walk_team(ngroups, MODE == 1 ? 8 : 2);
  const int wave = tid >> 6, lane = tid & 63, nwave = blockDim.x >> 6;
  // this half's first task of a group: tile ht % TQ, column ht / TQ
  auto prefetch = [&](long g) __attribute__((always_inline)) {
    const int ch = int(g / p.ngrp), t0 = int(g % p.ngrp) * TQ;
    if (ht < ntask1 && ht % TQ < min(TQ, tpc - t0)) fetch(ch, t0, ht % TQ, ht / TQ);
  };
  if (half == 0 && wk.g < wk.end) prefetch(wk.g);
  int turn = 0;  // the half whose columns are in registers for this group
  for (long g = wk.g; g < wk.end; g += wk.step, turn ^= 1) {
    const int ch = int(g / p.ngrp), t0 = int(g % p.ngrp) * TQ;
    const int nq = min(TQ, tpc - t0);
    const bool mine = half == turn;
    if (mine) {
      if (ht < ntask1 && ht % TQ < nq) column(ht % TQ, ht / TQ);
    } else {
      for (int k = HALF + ht; k < ntask1; k += HALF) {
        if (k % TQ >= nq) continue;
        fetch(ch, t0, k % TQ, k / TQ);
        column(k % TQ, k / TQ);
      }
    }
    __syncthreads();
    if (mine) {
      if (ht < ntask2 && ht % TQ < nq) rows(ht % TQ, (w0 + ht / TQ) & (H2 - 1));
    } else {
      for (int k = HALF + ht; k < ntask2; k += HALF)
        if (k % TQ < nq) rows(k % TQ, (w0 + k / TQ) & (H2 - 1));
      if (g + wk.step < wk.end) prefetch(g + wk.step);
    }
    __syncthreads();
    if (MODE == 1) {
      overlap_plane_out(p, ldf, TSZ, ch, t0, wave, lane, nwave);
    } else if (rot == 0) {
      crop(ch, t0, nq, wave, lane, nwave, std::false_type{});
    } else {
      crop(ch, t0, nq, wave, lane, nwave, std::true_type{});
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// overlap-add of tiles kept in the scratch (planes of more tiles than a
// workgroup holds): output pixel (i, j) of plane (img, ch) is the sum, in a
// fixed order, of the kept elements of the at most two tiles per side whose
// kept range covers framed pixel (i + off, j + off). A workgroup per (plane,
// run of rows), lanes over the columns.
__global__ void __launch_bounds__(256) overlap_gather_kernel(BigInvParams p, int rows_per_wg, int nrg) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned wg = xcd_local_order(blockIdx.x, gridDim.x);
  const int rg = int(wg % unsigned(nrg));
  const unsigned plane = wg / unsigned(nrg);
  const int img = int(plane / unsigned(p.n_ch)), ch = int(plane % unsigned(p.n_ch));
  const int H = p.H, T = p.T, b = p.pitch, KR = p.KR, P = T * T;
  const size_t tile_elems = size_t(KR) * KR;
  const float* tb = p.tiles + (size_t(ch) * p.n_img * P + size_t(img) * P) * tile_elems;
  float* out = p.dst + size_t(plane) * H * H;
  const SmallDiv div_b(b);
  const int i0 = rg * rows_per_wg, i1 = min(H, i0 + rows_per_wg);
  for (int i = i0 + wave; i < i1; i += 4) {
    const int a = i + p.off, P1 = div_b(a), ra1 = a - P1 * b;
    const bool r1 = P1 < T, r0 = P1 >= 1 && P1 - 1 < T && ra1 + b < KR;
    for (int jx = lane; jx < H; jx += 64) {
      const int c = jx + p.off, Q1 = div_b(c), ca1 = c - Q1 * b;
      const bool c1 = Q1 < T, c0 = Q1 >= 1 && Q1 - 1 < T && ca1 + b < KR;
      float acc = 0.f;
      if (r0 && c0) acc += tb[size_t((P1 - 1) * T + Q1 - 1) * tile_elems + (ra1 + b) * KR + ca1 + b];
      if (r0 && c1) acc += tb[size_t((P1 - 1) * T + Q1) * tile_elems + (ra1 + b) * KR + ca1];
      if (r1 && c0) acc += tb[size_t(P1 * T + Q1 - 1) * tile_elems + ra1 * KR + ca1 + b];
      if (r1 && c1) acc += tb[size_t(P1 * T + Q1) * tile_elems + ra1 * KR + ca1];
      out[size_t(i) * H + jx] = acc;
    }
  }
}

// ---------------------------------------------------------------------------
// launchers

// Waves of these kernels resident on a CU: every instance takes more than 128
// registers per lane, which leaves two waves on each of the four SIMDs.
constexpr int kBigWavesPerCu = 8;

// Persistent grid: whole rounds over the 8 XCDs, as many workgroups as are
// resident (by LDS and by registers), at most one per group.
unsigned persistent_grid(long ngroups, size_t lds, int nthr) {
  const long by_lds = long(kBigLds / std::max<size_t>(lds, 1));
  const long by_waves = kBigWavesPerCu / std::max(1, (nthr + 63) / 64);
  const long per_cu = std::max<long>(1, std::min(by_lds, by_waves));
  long nwg = std::min<long>(per_cu * device_cus(), (ngroups + 7) / 8 * 8);
  nwg = std::max<long>(8, nwg / 8 * 8);
  return unsigned(nwg);
}

// tiles per group: runs of eight (64-byte segments of a bin), or whole planes
// where fewer fit
int group_tiles(int P, long tpc) {
  int tq = OAA_BIG_TQ;
  if (P > 1 && P < tq) tq = P * (tq / P);
  return int(std::max<long>(1, std::min<long>(tq, tpc)));
}

// Forward tiles up to which L = 64 takes the kernels that spread a transform
// over lanes: one lane per transform needs about four groups of eight tiles
// per two CUs to overlap its halves. Measured: 100 tiles 6.4 against 13.7 us,
// 400 tiles 8.1 against 14.2, 2304 tiles 25.1 against 25.2, 27648 tiles 225
// against 208.
constexpr long kWideFwdTiles = 1536;
// The same for the inverse. Measured: crops of 100 tiles 7.9 against 11.1 us,
// 192 tiles of eight partial sums 28 against 43, 400 tiles 9.5 against 11.3,
// 1000 tiles 14.7 against 11.9; planes of one tile as the crops, planes of
// nine 23 against 17.
constexpr long kWideInvTiles = 512;

hipError_t launch_big_fwd(int L, BigFwdParams p, hipStream_t s) {
  if (p.S < 1 || p.S > L || p.T < 1 || p.H < 1 || size_t(p.H) * p.H * 4 >= (size_t(1) << 31))
    return hipErrorInvalidValue;
  const int P = p.T * p.T;
  const long tpc = long(p.n_img) * P;
  if (tpc < 1 || tpc > 0x7fffffffL) return hipErrorInvalidValue;
  if (p.run < 1) return hipErrorInvalidValue;
  if (L != Big::L || tpc * p.n_ch <= kWideFwdTiles) return launch_wide_rfft2(L, p, nullptr, s);
  p.TQ = group_tiles(P, tpc);
  p.ngrp = int((tpc + p.TQ - 1) / p.TQ);
  // one past the largest element the layout addresses
  const size_t end = size_t(Big::L * Big::V - 1) * p.bs + size_t(p.n_ch - 1) * p.cs +
                     size_t((tpc - 1) / p.run) * p.rs + size_t(std::min<long>(p.run, tpc));
  // the planes one group's windows read: tiles of at most TQ images
  const size_t span = (size_t(p.TQ - 1) * p.n_ch + 1) * size_t(p.H) * p.H * 4;
  const bool narrow = end * 8 < (size_t(1) << 32) && span < size_t(kOutOfRange);
  auto kern = narrow ? big_rfft2_lane_kernel<false> : big_rfft2_lane_kernel<true>;
  const hipError_t e = allow_lds(kern, kBigLds);
  if (e != hipSuccess) return e;
  const size_t lds = size_t(lane_tile_stride()) * p.TQ * 8;
  if (lds > kBigLds) return hipErrorInvalidConfiguration;
  constexpr int nthr = 512;  // two halves of four waves: 32 TQ <= 256 tasks per pass
  hipLaunchKernelGGL(kern, dim3(persistent_grid(long(p.n_ch) * p.ngrp, lds, nthr)), dim3(nthr), lds, s, p);
  return hipGetLastError();
}

// One sequence per lane, tiles of whole L x (L/2 + 1) slots
template <bool O32>
hipError_t launch_big_inv_lane_O(const BigInvParams& p, size_t lds, long ngroups, hipStream_t s) {
  void (*kern)(BigInvParams) = nullptr;
  if (p.overlap == 0)
    kern = p.nsplit > 1 ? big_irfft2_lane_kernel<O32, 0, true> : big_irfft2_lane_kernel<O32, 0, false>;
  else if (p.overlap == 1 && p.nsplit == 1)  // the overlap-add of forward spectra: one partial
    kern = big_irfft2_lane_kernel<O32, 1, false>;
  if (!kern) return hipErrorInvalidValue;
  const hipError_t e = allow_lds(kern, kBigLds);
  if (e != hipSuccess) return e;
  constexpr int nthr = 512;
  hipLaunchKernelGGL(kern, dim3(persistent_grid(ngroups, lds, nthr)), dim3(nthr), lds, s, p);
  return hipGetLastError();
}

hipError_t launch_big_inv_lane(const BigInvParams& p, long ngroups, hipStream_t s) {
  const size_t lds = size_t(lane_tile_stride()) * p.TQ * 8;
  if (lds > kBigLds || p.TQ > Big::TQ_MAX) return hipErrorInvalidConfiguration;
  const size_t tpc = size_t(p.n_img) * p.T * p.T;
  const bool o32 = (size_t(Big::L) * Big::V * size_t(p.n_ch) * tpc + size_t(p.nsplit - 1) * p.split_stride) * 8 <
                   (size_t(1) << 32);
  return o32 ? launch_big_inv_lane_O<true>(p, lds, ngroups, s) : launch_big_inv_lane_O<false>(p, lds, ngroups, s);
}

hipError_t launch_big_inv(int L, BigInvParams p, hipStream_t s) {
  if (p.KR < 1 || p.KR > L || p.rot < 0 || p.rot >= L || p.T < 1 || p.H < 1 || p.nsplit < 1 ||
      p.H >= 65536 || size_t(p.H) * p.H >= (size_t(1) << 31))
    return hipErrorInvalidValue;
  const int P = p.T * p.T;
  const long tpc = long(p.n_img) * P;
  if (tpc < 1 || tpc > 0x7fffffffL) return hipErrorInvalidValue;
  bool two_step = false;
  if (p.overlap) {
    if (p.pitch < 1 || p.off < 0 || p.H + p.off >= 65536 || p.nsplit != 1) return hipErrorInvalidValue;
    if (!p.tiles && big_overlap_few(L, long(p.n_img) * p.n_ch, p.T)) {
      p.overlap = 3;
      return launch_wide_irfft2(L, p, s);
    }
    if (!big_overlap_supported(L, p.T)) {
      // side 128: keep every tile's KR x KR in the scratch, then add in a second kernel
      if (L == Big::L || !p.tiles || long(p.KR) * p.KR >= 65536) return hipErrorInvalidValue;
      two_step = true;
      p.overlap = 2;
    }
  } else if (p.pitch != p.KR) {
    return hipErrorInvalidValue;
  }
  hipError_t e = hipSuccess;
  if (L != Big::L || (tpc * p.n_ch <= kWideInvTiles && (p.overlap != 1 || P == 1))) {
    e = launch_wide_irfft2(L, p, s);
  } else {
    p.TQ = p.overlap == 1 ? P : group_tiles(P, tpc);  // overlap-add in a group: one plane
    if (!p.overlap && long(p.KR) * p.KR * p.TQ >= 65536) return hipErrorInvalidValue;
    p.ngrp = int((tpc + p.TQ - 1) / p.TQ);
    e = launch_big_inv_lane(p, long(p.n_ch) * p.ngrp, s);
  }
  if (e != hipSuccess || !two_step) return e;
  // second step: about 8 rows per workgroup
  const int rows = 8, nrg = (p.H + rows - 1) / rows;
  const long nwg = long(p.n_img) * p.n_ch * nrg;
  if (nwg > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(overlap_gather_kernel, dim3(unsigned(nwg)), dim3(256), 0, s, p, rows, nrg);
  return hipGetLastError();
}

}  // namespace

int device_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    cached[dev] = cus;
  }
  return cached[dev];
}

hipError_t launch_big_rfft2(int L, const BigFwdParams& p, hipStream_t s) {
  return L == 64 || L == 128 ? launch_big_fwd(L, p, s) : hipErrorInvalidValue;
}

hipError_t launch_big_irfft2(int L, const BigInvParams& p, hipStream_t s) {
  return L == 64 || L == 128 ? launch_big_inv(L, p, s) : hipErrorInvalidValue;
}

// The block-by-block kernel inverts each tile four times, the one with a
// workgroup per block row about three: it pays while its blocks are at most
// one per CU. Measured, with the stage's events: one 224 x 224 plane of 16
// tiles 15 against 25 us, 256 tiles 17 against 26, 512 tiles 28 against 26,
// 1024 tiles 51 against 32.
bool big_overlap_few(int L, long n_planes, int T) {
  return L == 64 && !big_overlap_supported(L, T) && n_planes * T * T <= 256;
}

bool big_overlap_supported(int L, int T) {
  // whole tiles in LDS: nine of side 64, one of side 128
  return L == 64 ? T <= Big::SIDE_MAX : L == 128 && T == 1;
}

}  // namespace oaa
