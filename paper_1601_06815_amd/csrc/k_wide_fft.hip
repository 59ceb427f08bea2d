// Transforms of side L = 128, and of sides 16 to 64 in launches of few tiles
// or in the shapes that the other kernels serve less well (wide_takes,
// wide_overlap, wide_pair_fits) (arXiv:1601.06815, Section 2: block division,
// zero padding, the per-block transforms and the overlap-add; Section 3.3 for
// the transform sides of large kernels), with each L-point transform spread
// over lanes.
//
// L = N1 x 8 (4 x 4 at L = 16). With n = 8 n1 + n2 and k = k1 + N1 k2,
//   X[k1 + N1 k2] = sum_n2 w8^(n2 k2) ( wL^(n2 k1) sum_n1 wN1^(n1 k1) x[8 n1 + n2] ),
// so a transform takes two passes over LDS: N1-point transforms over the
// elements of one n2 with a twiddle, then 8-point transforms over n2. Both
// passes read and write the same slots of a sequence, and coefficient k ends
// at position 8 (k mod N1) + k / N1 (`place`). A tile's 2-D transform is four
// such passes, on 8 L/2 tasks of N1 points and N1 L/2 tasks of 8 points: one
// tile keeps 8 (L = 128) waves busy in about 60 registers, and the chain that
// a lane runs is short. What bounds a launch of few tiles is that chain.
// Transforms held by lane pairs (64 points per lane and pass, 256 registers
// with 600 bytes of them spilled at L = 128, two waves per tile) took 62 us for
// the forward inverse of 100 tiles of 128 x 128 and 45 us for the one tile of
// the error propagation, now 23 and 16; and 3.8 ms for 16384 tiles, now 1.5.
#include <algorithm>

#include "fft_core.hpp"
#include "oaa_internal.hpp"
#include "tile_common.hpp"

namespace oaa {

namespace {

using namespace tile;

constexpr size_t kWideLds = 160 * 1024;  // LDS of one CU
constexpr int kWideMaxThreads = 1024;
constexpr long kWideTiles = 1536;  // tiles of a launch of few

template <int L>
struct Wide {
  static constexpr int N2 = L == 16 ? 4 : 8, N1 = L / N2, H2 = L / 2, V = L / 2 + 1;
  static constexpr int RS = H2 + 1;          // LDS row stride (complex)
  static constexpr int TS = L * RS | 1;      // LDS per tile (complex, odd)
  static constexpr int TASKS = N2 * H2;      // N1-point tasks of a pass
  static constexpr int TASKS2 = N1 * H2;     // N2-point tasks of a pass
  __device__ static constexpr int place(int k) { return N2 * (k % N1) + k / N1; }
};

// (re + i im) w_L^(SIGN n2 k1), w_L from the table of cosines and sines in LDS
template <int L, int SIGN>
__device__ __forceinline__ float2 turned(const float2* tw, int n2, int k1, float re, float im) {
  if (k1 == 0) return make_float2(re, im);
  const float2 w = tw[n2 * k1];
  const float s = SIGN > 0 ? w.y : -w.y;
  return make_float2(__builtin_fmaf(re, w.x, -im * s), __builtin_fmaf(re, s, im * w.x));
}

// cos and sin of 2 pi k / L, k < L, into LDS
template <int L>
__device__ __forceinline__ void load_twiddles(float2* tw) {
  for (int k = threadIdx.x; k < L; k += blockDim.x) tw[k] = make_float2(tw::kTable<L>.c[k], tw::kTable<L>.s[k]);
}

// N2-point pass over n2 of the sequence element (k1, n2) at z[(N2 k1 + n2) stride]
template <int N2, int SIGN>
__device__ __forceinline__ void pass2(float2* z, int stride) {
  float re[N2], im[N2];
#pragma unroll
  for (int i = 0; i < N2; ++i) {
    const float2 v = z[i * stride];
    re[i] = v.x;
    im[i] = v.y;
  }
  fft_dif<N2, SIGN, false>(re, im);
#pragma unroll
  for (int k = 0; k < N2; ++k) z[k * stride] = make_float2(re[bitrev(k, N2)], im[bitrev(k, N2)]);
}

// ---------------------------------------------------------------------------
// forward: windows of planes -> half spectra
//
// Columns: z = x[., j] + i x[., j + L/2] along the rows; the real columns'
// spectra are C_j[u] = (Z[u] + conj Z[-u]) / 2 and C_{j+L/2}[u] =
// (Z[u] - conj Z[-u]) / (2i), taken as the row pass reads them. Rows: row u in
// [1, L/2) along the columns gives bins (u, v), v <= L/2, and (L - u, v) =
// conj X[u][L - v], 0 < v < L/2 (the other bins of rows past L/2 are
// conjugates that nothing reads); it uses the storage of LDS rows u and L - u.
// Rows 0 and L/2 are real and go through one transform as row 0.
//
// A launch does one job or two (kernel and input spectra), whose groups follow
// one another: each launch of these sizes costs about as long as its work.
// Up to L = 32 the bins of rows past L/2 in columns 0 and L/2 are written too,
// as by the kernels of many tiles.
template <int L>
__global__ void __launch_bounds__(kWideMaxThreads) wide_rfft2_kernel(BigFwdParams pa, BigFwdParams pb) {
  using W = Wide<L>;
  constexpr int N1 = W::N1, N2 = W::N2, H2 = W::H2, V = W::V, RS = W::RS;
  extern __shared__ float smem[];
  float2* tw = reinterpret_cast<float2*>(smem);
  float2* lds = tw + L;
  const int tid = threadIdx.x, nthr = blockDim.x, TQ = pa.TQ;
  const long na = long(pa.n_ch) * pa.ngrp, ngroups = na + long(pb.n_ch) * pb.ngrp;
  load_twiddles<L>(tw);
  __syncthreads();
  for (long gg = long(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8; gg < ngroups; gg += gridDim.x) {
    const BigFwdParams& p = gg < na ? pa : pb;
    const long g = gg < na ? gg : gg - na;
    const int P = p.T * p.T, tpc = p.n_img * P;
    const size_t bs = p.bs;
    const int ch = int(g / p.ngrp), t0 = int(g % p.ngrp) * TQ;
    const int nq = min(TQ, tpc - t0);
    // columns, N1 points: lanes over the columns (a wave holds one tile)
    for (int task = tid; task < nq * W::TASKS; task += nthr) {
      const int j = task % H2, n2 = (task / H2) % N2, q = task / W::TASKS;
      const int t = t0 + q, img = t / P, pp = t - img * P;
      const int pr = pp / p.T, qc = pp - pr * p.T;
      const float* plane = p.src + (size_t(img) * p.n_ch + ch) * size_t(p.H) * size_t(p.H);
      const int ca = qc * p.pitch - p.off + j, cb = ca + H2, gr0 = pr * p.pitch - p.off + n2;
      const bool oka = j < p.S && unsigned(ca) < unsigned(p.H);
      const bool okb = j + H2 < p.S && unsigned(cb) < unsigned(p.H);
      float re[N1], im[N1];
      if constexpr (W::TASKS % 64 == 0) {
        const __amdgpu_buffer_rsrc_t rs = buffer_resource(plane, unsigned(p.H) * unsigned(p.H) * 4u);
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          const int gr = gr0 + N2 * i;
          const bool okr = N2 * i + n2 < p.S && unsigned(gr) < unsigned(p.H);
          re[i] = buffer_load_f1(rs, okr && oka ? unsigned(gr * p.H + ca) * 4u : kOutOfRange);
          im[i] = buffer_load_f1(rs, okr && okb ? unsigned(gr * p.H + cb) * 4u : kOutOfRange);
        }
      } else {  // two tiles per wave, perhaps of two planes: clamped addresses
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          const int gr = gr0 + N2 * i;
          const bool okr = N2 * i + n2 < p.S && unsigned(gr) < unsigned(p.H);
          const float a = plane[okr && oka ? gr * p.H + ca : 0], c = plane[okr && okb ? gr * p.H + cb : 0];
          re[i] = okr && oka ? a : 0.f;
          im[i] = okr && okb ? c : 0.f;
        }
      }
      fft_dif<N1, -1, false>(re, im);
      float2* z = lds + q * W::TS + n2 * RS + j;
#pragma unroll
      for (int k = 0; k < N1; ++k)
        z[N2 * k * RS] = turned<L, -1>(tw, n2, k, re[bitrev(k, N1)], im[bitrev(k, N1)]);
    }
    __syncthreads();
    // columns, 8 points
    for (int task = tid; task < nq * W::TASKS2; task += nthr) {
      const int j = task % H2, k1 = (task / H2) % N1, q = task / W::TASKS2;
      pass2<N2, -1>(lds + q * W::TS + N2 * k1 * RS + j, RS);
    }
    __syncthreads();
    // rows, N1 points: lanes over n2, then the rows
    for (int task = tid; task < nq * W::TASKS; task += nthr) {
      const int n2 = task % N2, u = (task / N2) % H2, q = task / W::TASKS;
      float2* za = lds + q * W::TS + W::place(u) * RS + n2;
      float2* zb = lds + q * W::TS + W::place(u ? L - u : H2) * RS + n2;
      float re[N1], im[N1];
#pragma unroll
      for (int i = 0; i < N1 / 2; ++i) {
        const float2 a = za[N2 * i], c = zb[N2 * i];
        re[i] = u ? 0.5f * (a.x + c.x) : a.x;
        im[i] = u ? 0.5f * (a.y - c.y) : c.x;
        re[N1 / 2 + i] = u ? 0.5f * (a.y + c.y) : a.y;
        im[N1 / 2 + i] = u ? 0.5f * (c.x - a.x) : c.y;
      }
      fft_dif<N1, -1, false>(re, im);
#pragma unroll
      for (int k = 0; k < N1 / 2; ++k) {
        za[N2 * k] = turned<L, -1>(tw, n2, k, re[bitrev(k, N1)], im[bitrev(k, N1)]);
        zb[N2 * k] = turned<L, -1>(tw, n2, k + N1 / 2, re[bitrev(k + N1 / 2, N1)], im[bitrev(k + N1 / 2, N1)]);
      }
    }
    __syncthreads();
    // rows, 8 points, and the bins: lanes over the group's tiles, then the rows
    for (int task = tid; task < TQ * W::TASKS2; task += nthr) {
      const int q = task % TQ, u = (task / TQ) % H2, k1 = task / (TQ * H2);
      if (q >= nq) continue;
      float2* z = lds + q * W::TS + W::place(k1 < N1 / 2 ? u : u ? L - u : H2) * RS + N2 * (k1 % (N1 / 2));
      if (u == 0) {  // the packed row stays in LDS
        pass2<N2, -1>(z, 1);
        continue;
      }
      float re[N2], im[N2];
#pragma unroll
      for (int i = 0; i < N2; ++i) {
        re[i] = z[i].x;
        im[i] = z[i].y;
      }
      fft_dif<N2, -1, false>(re, im);
      const int t = t0 + q;
      float2* out = p.dst + size_t(ch) * p.cs + size_t(t / p.run) * p.rs + size_t(t % p.run);
      float2* o1 = out + (size_t(u) * V + k1) * bs;            // (u, k1 + N1 k2)
      float2* o2 = out + (size_t(L - u) * V + L - k1) * bs;    // (L - u, L - k1 - N1 k2)
#pragma unroll
      for (int k = 0; k < N2; ++k) {
        const float r = re[bitrev(k, N2)], i = im[bitrev(k, N2)];
        if (k < N2 / 2 || (k == N2 / 2 && k1 == 0)) {
          o1[size_t(k * N1) * bs] = make_float2(r, i);
          if (L <= 32 && (k == 0 || k == N2 / 2) && k1 == 0)  // column 0 or L/2
            out[(size_t(L - u) * V + k * N1) * bs] = make_float2(r, -i);
        } else {
          *(o2 - size_t(k * N1) * bs) = make_float2(r, -i);
        }
      }
    }
    __syncthreads();
    // the packed row gives rows 0 and L/2
    for (int task = tid; task < TQ * V; task += nthr) {
      const int q = task % TQ, v = task / TQ;
      if (q >= nq) continue;
      const float2* z0 = lds + q * W::TS + W::place(0) * RS;
      const float2* z1 = lds + q * W::TS + W::place(H2) * RS;
      auto at = [&](int k) {
        const int pos = W::place(k);
        return pos < H2 ? z0[pos] : z1[pos - H2];
      };
      const float2 a = at(v), c = at((L - v) % L);
      const int t = t0 + q;
      float2* out = p.dst + size_t(ch) * p.cs + size_t(t / p.run) * p.rs + size_t(t % p.run);
      // halved before they are added: the sums of bins past 1.7e38 would overflow
      out[size_t(v) * bs] = make_float2(0.5f * a.x + 0.5f * c.x, 0.5f * a.y - 0.5f * c.y);
      out[(size_t(H2) * V + v) * bs] = make_float2(0.5f * a.y + 0.5f * c.y, 0.5f * c.x - 0.5f * a.x);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// inverse: half spectra -> kept part of every tile (crop), or the plane the
// tiles overlap-add to
//
// Columns w < L/2 along u; column 0 carries the real columns 0 and L/2
// together as h0[u] + i h1[u] (rows past L/2 rebuilt as the conjugates of rows
// L - u, which are not stored). Then pairs of kept rows as one complex
// sequence, in the storage of the pair's two LDS rows. Rows and columns stay at
// their inverse index, kept index (r + rot) mod L; the output pass scales.
// MODE: 0 crop, 1 overlap-add of planes whose tiles fit the group, 2 tiles to
// the scratch, 3 overlap-add by output block: a group is block (P, Q) of a
// plane, To x To blocks per plane, and its tiles the four that reach the block,
// (P - 1 + q / 2, Q - 1 + q % 2), each block's tiles inverted anew. Every sum
// is taken in a fixed order.
template <int L, int MODE>
__global__ void __launch_bounds__(kWideMaxThreads) wide_irfft2_kernel(BigInvParams p) {
  using W = Wide<L>;
  constexpr int N1 = W::N1, N2 = W::N2, H2 = W::H2, V = W::V, RS = W::RS;
  extern __shared__ float smem[];
  float2* tw = reinterpret_cast<float2*>(smem);
  float2* lds = tw + L;
  const float* ldf = reinterpret_cast<const float*>(lds);
  const int tid = threadIdx.x, nthr = blockDim.x, TQ = p.TQ;
  const int KR = p.KR, rot = p.rot, npair = (KR + 1) / 2;
  const int P = p.T * p.T, tpc = p.n_img * P;
  const size_t fstride = size_t(p.n_ch) * tpc;
  const long ngroups = long(p.n_ch) * p.ngrp;
  const float scale = 1.0f / float(L * L);
  // inverse index of kept index k
  auto inverse = [&](int k) { return (k - rot) & (L - 1); };
  load_twiddles<L>(tw);
  __syncthreads();
  for (long g = long(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8; g < ngroups; g += gridDim.x) {
    const int ch = int(g / p.ngrp);
    // MODE 3: output block (Pb, Qb) of image t0 / P
    const int blk = int(g % p.ngrp), To = p.To, Pb = MODE == 3 ? blk / To % To : 0, Qb = MODE == 3 ? blk % To : 0;
    const int t0 = MODE == 3 ? blk / (To * To) * P : blk * TQ;
    const int nq = MODE == 3 ? 4 : min(TQ, tpc - t0);
    // tile q of the group, and whether there is one
    auto tile_at = [&](int q) {
      return MODE == 3 ? t0 + (Pb - 1 + q / 2) * p.T + Qb - 1 + q % 2 : t0 + q;
    };
    auto has = [&](int q) {
      return MODE == 3 ? unsigned(Pb - 1 + q / 2) < unsigned(p.T) && unsigned(Qb - 1 + q % 2) < unsigned(p.T) : q < nq;
    };
    // columns, N1 points: lanes over the group's tiles, then the columns;
    // column 0 last, so that its other arithmetic meets one wave only
    for (int task = tid; task < TQ * W::TASKS; task += nthr) {
      const int q = task % TQ, rest = task / TQ;
      if (!has(q)) continue;
      const bool edge = rest >= N2 * (H2 - 1);
      const int w = edge ? 0 : 1 + rest % (H2 - 1), n2 = edge ? rest - N2 * (H2 - 1) : rest / (H2 - 1);
      const float2* src = p.src + size_t(ch) * tpc + tile_at(q);
      float re[N1], im[N1];
#pragma unroll
      for (int i = 0; i < N1; ++i) re[i] = im[i] = 0.f;
      // addresses step from an opaque pointer, so that those of all elements
      // are not held at once
      const size_t step = size_t(N2 * V) * fstride;
      for (int sp = 0; sp < p.nsplit; ++sp) {
        const float2* b = src + size_t(sp) * p.split_stride + (size_t(n2) * V + w) * fstride;
        asm volatile("" : "+v"(b));
        if (!edge) {
#pragma unroll
          for (int i = 0; i < N1; ++i, b += step) {
            const float2 z = *b;
            re[i] += z.x;
            im[i] += z.y;
          }
        } else {
#pragma unroll
          for (int i = 0; i < N1; ++i) {
            // rows up to L/2, then L - u for the rows u = N2 i + n2 past it
            if (i == N1 / 2 && n2 != 0) b -= size_t(2 * n2) * V * fstride;
            const bool mirror = i > N1 / 2 || (i == N1 / 2 && n2 != 0);
            const float2 b0 = b[0], b1 = b[size_t(H2) * fstride];
            re[i] += mirror ? b0.x + b1.y : b0.x - b1.y;
            im[i] += mirror ? b1.x - b0.y : b0.y + b1.x;
            if (i < N1 / 2) b += step; else b -= step;
          }
        }
      }
      fft_dif<N1, +1, false>(re, im);
      float2* z = lds + q * W::TS + n2 * RS + w;
#pragma unroll
      for (int k = 0; k < N1; ++k)
        z[N2 * k * RS] = turned<L, +1>(tw, n2, k, re[bitrev(k, N1)], im[bitrev(k, N1)]);
    }
    __syncthreads();
    // columns, 8 points
    for (int task = tid; task < nq * W::TASKS2; task += nthr) {
      const int w = task % H2, k1 = (task / H2) % N1, q = task / W::TASKS2;
      pass2<N2, +1>(lds + q * W::TS + N2 * k1 * RS + w, RS);
    }
    __syncthreads();
    // row pairs, N1 points: lanes over n2, then the pairs. A task reads the
    // slots of n2 and of N2 - n2, which another lane of the same N2 writes:
    // all read before any writes.
    const int ntask = nq * npair * N2;
    for (int base = 0; base < ntask; base += nthr) {
      const int task = base + tid;
      const bool live = task < ntask;
      const int n2 = task % N2, pair = live ? (task / N2) % npair : 0, q = live ? task / (N2 * npair) : 0;
      float2* za = lds + q * W::TS + W::place(inverse(2 * pair)) * RS;
      float2* zb = lds + q * W::TS + W::place(inverse(2 * pair + 1)) * RS;
      const bool has1 = 2 * pair + 1 < KR;
      float re[N1], im[N1];
      if (live) {
#pragma unroll
        for (int i = 0; i < N1 / 2; ++i) {
          const int v = N2 * i + n2, m = H2 - v;  // element v, and element L/2 + v from bin m
          float2 a = za[v], b = has1 ? zb[v] : make_float2(0.f, 0.f);
          const bool first = v == 0;  // bins 0 and L/2 are the parts of slot 0
          re[i] = first ? a.x : a.x - b.y;
          im[i] = first ? b.x : a.y + b.x;
          const float2 c = za[first ? 0 : m], d = has1 ? zb[first ? 0 : m] : make_float2(0.f, 0.f);
          re[N1 / 2 + i] = first ? a.y : c.x + d.y;
          im[N1 / 2 + i] = first ? b.y : d.x - c.y;
        }
        fft_dif<N1, +1, false>(re, im);
      }
      __syncthreads();
      if (live) {
#pragma unroll
        for (int k = 0; k < N1 / 2; ++k) {
          za[N2 * k + n2] = turned<L, +1>(tw, n2, k, re[bitrev(k, N1)], im[bitrev(k, N1)]);
          zb[N2 * k + n2] = turned<L, +1>(tw, n2, k + N1 / 2, re[bitrev(k + N1 / 2, N1)], im[bitrev(k + N1 / 2, N1)]);
        }
      }
    }
    __syncthreads();
    // row pairs, 8 points
    for (int task = tid; task < nq * npair * N1; task += nthr) {
      const int pair = task % npair, k1 = (task / npair) % N1, q = task / (npair * N1);
      const int row = inverse(2 * pair + (k1 < N1 / 2 ? 0 : 1));
      pass2<N2, +1>(lds + q * W::TS + W::place(row) * RS + N2 * (k1 % (N1 / 2)), 1);
    }
    __syncthreads();
    // real element at kept row a, kept column c of tile q, unscaled
    auto row_base = [&](int q, int a, int& second) {
      second = (W::place(inverse(a | 1)) - W::place(inverse(a & ~1))) * RS * 2;
      return (q * W::TS + W::place(inverse(a & ~1)) * RS) * 2 + (a & 1);
    };
    auto at = [&](int rb, int second, int c) {
      const int pos = W::place(inverse(c));
      return ldf[rb + (pos < H2 ? 2 * pos : second + 2 * (pos - H2))];
    };
    const int H = p.H, lane = tid & 63, wave = tid >> 6, nwave = nthr >> 6;
    if (MODE == 3) {
      // rows and columns of the block inside the plane: a wave per row
      const int img = t0 / P, b = p.pitch, i0 = Pb * b - p.off, j0 = Qb * b - p.off;
      float* out = p.dst + (size_t(img) * p.n_ch + ch) * H * H;
      for (int r = max(0, -i0) + wave; r < min(b, H - i0); r += nwave) {
        for (int c = max(0, -j0) + lane; c < min(b, H - j0); c += 64) {
          float acc = 0.f;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int a = q / 2 ? r : r + b, cc = q % 2 ? c : c + b;
            if (!has(q) || a >= KR || cc >= KR) continue;
            int second;
            const int rb = row_base(q, a, second);
            acc = __builtin_fmaf(scale, at(rb, second, cc), acc);
          }
          out[size_t(i0 + r) * H + j0 + c] = acc;
        }
      }
    } else if (MODE == 1) {
      // plane = group: a wave per output row, lanes over the columns
      const int img = t0 / P, T = p.T, b = p.pitch;
      float* out = p.dst + (size_t(img) * p.n_ch + ch) * H * H;
      const SmallDiv div_b(b);
      for (int i = wave; i < H; i += nwave) {
        const int a = i + p.off, P1 = div_b(a), ra1 = a - P1 * b;
        const bool r1 = P1 < T, r0 = P1 >= 1 && P1 - 1 < T && ra1 + b < KR;
        for (int jx = lane; jx < H; jx += 64) {
          const int c = jx + p.off, Q1 = div_b(c), ca1 = c - Q1 * b;
          const bool c1 = Q1 < T, c0 = Q1 >= 1 && Q1 - 1 < T && ca1 + b < KR;
          float acc = 0.f;
          auto add = [&](bool on, int Pt, int Qt, int ra, int ca) {
            if (!on) return;
            int second;
            const int rb = row_base(Pt * T + Qt, ra, second);
            acc = __builtin_fmaf(scale, at(rb, second, ca), acc);
          };
          add(r0 && c0, P1 - 1, Q1 - 1, ra1 + b, ca1 + b);
          add(r0 && c1, P1 - 1, Q1, ra1 + b, ca1);
          add(r1 && c0, P1, Q1 - 1, ra1, ca1 + b);
          add(r1 && c1, P1, Q1, ra1, ca1);
          out[size_t(i) * H + jx] = acc;
        }
      }
    } else {
      // a wave per kept row of a tile, lanes over its columns
      for (int r = wave; r < nq * KR; r += nwave) {
        const int q = r / KR, a = r - q * KR, t = t0 + q;
        int second;
        const int rb = row_base(q, a, second);
        if (MODE == 2) {
          float* ot = p.tiles + ((size_t(ch) * tpc + t) * KR + a) * KR;
          for (int c = lane; c < KR; c += 64) ot[c] = at(rb, second, c) * scale;
        } else {
          const int img = t / P, pp = t - img * P, pr = pp / p.T, qc = pp - pr * p.T;
          if (pr * p.pitch + a >= H) continue;
          const int ncol = min(KR, H - qc * p.pitch);
          float* orow = p.dst + ((size_t(img) * p.n_ch + ch) * H + pr * p.pitch + a) * H + qc * p.pitch;
          for (int c = lane; c < ncol; c += 64) orow[c] = at(rb, second, c) * scale;
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// launchers

template <int L>
constexpr size_t wide_lds(int TQ) { return (size_t(Wide<L>::TS) * TQ + L) * 8; }

// Threads: one N1-point task each, in whole waves (the output passes step by
// waves), up to a whole workgroup.
template <int L>
int wide_threads(int TQ) { return std::min(kWideMaxThreads, (Wide<L>::TASKS * TQ + 63) / 64 * 64); }

// Persistent grid: as many workgroups as are resident (by LDS; two of 512 or
// one of 1024 lanes by registers), whole rounds over the 8 XCDs.
template <int L>
unsigned wide_grid(long ngroups, int TQ) {
  const long per_cu = std::max<long>(1, std::min<long>(long(kWideLds / wide_lds<L>(TQ)), 1024 / wide_threads<L>(TQ)));
  return unsigned(std::max<long>(8, std::min<long>(per_cu * device_cus(), (ngroups + 7) / 8 * 8) / 8 * 8));
}

// Tiles per group: one while they are at most one per CU, then more, for
// longer runs of a bin and fewer barriers per tile. Measured at L = 128: forward
// 400 tiles 28 us one by one and 22 in pairs, 16384 tiles 1.91 and 1.08 ms;
// inverse 400 tiles 33 and 27 us, but 4096 tiles 0.36 and 0.41 ms (a pair
// leaves one workgroup per CU). At L = 32, forward: 49 tiles 4.3 us one by one
// and 4.9 in fours, 855 tiles 6.8 and 5.6 (8.4 in sixteens), 6912 tiles 31, 21
// and 17, 147456 tiles 861, 398 and 268.
template <int L>
int wide_tiles(long tiles, long tpc, bool inverse) {
  if (tpc < 2 || tiles <= device_cus()) return 1;
  if (L <= 32) return int(std::min<long>(tpc, tiles <= kWideTiles ? 4 : 16));
  return inverse && tiles > kWideTiles ? 1 : 2;
}

template <int L>
hipError_t launch_fwd(BigFwdParams a, BigFwdParams b, bool two, hipStream_t s) {
  const long ta = long(a.n_img) * a.T * a.T, tb = two ? long(b.n_img) * b.T * b.T : 0;
  const long tiles = ta * a.n_ch + (two ? tb * b.n_ch : 0);
  a.TQ = b.TQ = wide_tiles<L>(tiles, std::max(ta, tb), false);
  a.ngrp = int((ta + a.TQ - 1) / a.TQ);
  b.ngrp = int((tb + b.TQ - 1) / b.TQ);
  auto kern = wide_rfft2_kernel<L>;
  const hipError_t e = allow_lds(kern, kWideLds);
  if (e != hipSuccess) return e;
  const long groups = long(a.n_ch) * a.ngrp + long(b.n_ch) * b.ngrp;
  hipLaunchKernelGGL(kern, dim3(wide_grid<L>(groups, a.TQ)), dim3(wide_threads<L>(a.TQ)), wide_lds<L>(a.TQ), s, a, b);
  return hipGetLastError();
}

template <int L, int MODE>
hipError_t launch_inv_mode(BigInvParams p, hipStream_t s) {
  const long tpc = long(p.n_img) * p.T * p.T;
  p.TQ = MODE == 1 ? p.T * p.T : MODE == 3 ? 4 : wide_tiles<L>(tpc * p.n_ch, tpc, true);
  p.To = MODE == 3 ? (p.H + p.off + p.pitch - 1) / p.pitch : 0;
  const long groups = MODE == 3 ? long(p.n_img) * p.To * p.To : (tpc + p.TQ - 1) / p.TQ;
  if (groups > 0x7fffffffL || (MODE == 3 && (p.To < p.T || p.KR > 2 * p.pitch))) return hipErrorInvalidValue;
  p.ngrp = int(groups);
  if (wide_lds<L>(p.TQ) > kWideLds) return hipErrorInvalidConfiguration;
  auto kern = wide_irfft2_kernel<L, MODE>;
  const hipError_t e = allow_lds(kern, kWideLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(wide_grid<L>(long(p.n_ch) * p.ngrp, p.TQ)), dim3(wide_threads<L>(p.TQ)),
                     wide_lds<L>(p.TQ), s, p);
  return hipGetLastError();
}

// The modes that a side is asked for: at 32 the overlap-adds (wide_overlap)
// only, its crops being the other kernels'; the scratch at 128 only, whose
// planes of several tiles have no other kernel.
template <int L>
hipError_t launch_inv(const BigInvParams& p, hipStream_t s) {
  if (p.overlap == 1) return launch_inv_mode<L, 1>(p, s);
  if constexpr (L <= 64) {
    if (p.overlap == 3) return launch_inv_mode<L, 3>(p, s);
  }
  if constexpr (L >= 64) {
    if (p.overlap == 0) return launch_inv_mode<L, 0>(p, s);
  }
  if constexpr (L == 128) {
    if (p.overlap == 2) return launch_inv_mode<L, 2>(p, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Few enough planes of few enough bytes for the 32-bit offsets of the loads.
static bool plane_fits(int H) { return size_t(H) * H * 4 < (size_t(1) << 31); }

bool wide_pair_fits(int L, long tiles_a, int Ha, long tiles_b, int Hb) {
  return L >= 16 && tiles_a + tiles_b <= kWideTiles && plane_fits(Ha) && plane_fits(Hb);
}

bool wide_takes(int L, WideUse use, long tiles, int T, int H) {
  if (L != 32 || !plane_fits(H)) return false;
  switch (use) {
    case WideUse::kernels: return tiles <= 1024;
    case WideUse::blocks: return tiles <= kWideTiles || T < 16;
    default: return tiles <= kWideTiles || (tiles >= 32768 && 16 % T != 0);
  }
}

int wide_overlap(int L, long n_planes, int T, int b) {
  if (L != 32) return 0;
  if (n_planes * T * T <= 256) return 3;
  return T <= 4 && 2 * b > L && n_planes <= 4096 ? 1 : 0;
}

hipError_t launch_wide_rfft2(int L, const BigFwdParams& a, const BigFwdParams* b, hipStream_t s) {
  BigFwdParams pb{};
  if (b) pb = *b;
  pb.T = std::max(pb.T, 1);
  switch (L) {
    case 16: return launch_fwd<16>(a, pb, b != nullptr, s);
    case 32: return launch_fwd<32>(a, pb, b != nullptr, s);
    case 64: return launch_fwd<64>(a, pb, b != nullptr, s);
    case 128: return launch_fwd<128>(a, pb, b != nullptr, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_wide_irfft2(int L, const BigInvParams& p, hipStream_t s) {
  switch (L) {
    case 32: return launch_inv<32>(p, s);
    case 64: return launch_inv<64>(p, s);
    case 128: return launch_inv<128>(p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace oaa
