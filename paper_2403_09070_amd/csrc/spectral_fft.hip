// Fast transforms for the spectral Poisson solve (Sec. III-A, Eqs. density-coef,
// poisson-sol-potential, possion-sol-force) on grids whose planar sides are powers of two and
// whose Nz is 2 or 4: the same cosine / sine series as the dense contractions, in float32, with
// N log N operations per row instead of N^2.
//
// A cosine row transform is a complex FFT of the row's even samples followed by its odd samples
// backwards (Makhoul, "A fast cosine transform in one and two dimensions", 1980), and two real
// rows share one complex FFT.  With Z the FFT of v_a + i v_b and m = N - k,
//   V_a(k) = (Z_k + conj Z_m) / 2,  V_b(k) = (Z_k - conj Z_m) / 2i,  w_k = e^{-i pi k / 2N},
//   w_k V(k) = X_k - i X_m                     (X the unnormalised cosine sums of one row)
// so that one pair (k, m) of FFT outputs gives both coefficients of both rows; and the inverse row
// of coefficients b starts from
//   V'(k) = conj(w_k) (b_k - i b_m) / 2,  V'(m) = conj V'(k),  V'(0) = b_0,
// whose inverse FFT holds the samples in the same order.  The sine series is the cosine series of
// the reversed coefficients with every odd sample negated: sin(pi k (n + 1/2) / N) =
// (-1)^n cos(pi (N - k)(n + 1/2) / N).
//
// Three launches:
//   k_fft_x    rho rows (two rows y, y + 1 per FFT) -> t[x frequency][z][y]
//   k_fft_y    per x frequency, all layers: forward y, z mixing and 1 / |omega|^2, inverse y (cosine
//              -> vg, sine -> vh), [x frequency / 2][y][z frequency][2]
//   k_fft_ix   per row y and output map: z mixing, inverse x, the map's rows in natural order
//
// An FFT of N points is held by a group of T = N / E lanes, E points in each lane's registers: lane t
// holds points t + T s.  Three radix stages (16 x 8 x 8 at N = 1024) with two exchanges through LDS;
// up to N = 1024 a group's lanes are of one wavefront, so that no workgroup barrier stands inside a
// transform.  An index i of a buffer sits at i + i / 16, which keeps the strided writes of a stage
// on distinct banks.
//
// What bounds them: at 1024 x 1024 x 4 the kernels move 34, 50 and 84 MB in 11, 21 and 22 us (3.1,
// 2.4 and 3.8 TB/s against 5.1 for a copy); their vector instructions alone take about 3, 10 and 9 us,
// and two or three wavefronts per SIMD, the registers' and the grid's limit, leave the LDS and load
// latencies of their one or two rounds in sight.  The four dense split contractions and the fold
// they replace take 143 us, the float32 ones with their z passes 418 us.
#include <cmath>

#include "internal.h"

namespace p3d {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
struct cf { float x, y; };
__device__ __forceinline__ cf operator+(cf a, cf b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cf operator-(cf a, cf b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cf cmul(cf a, cf b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ cf conj_mul(cf w, cf b) { return {w.x * b.x + w.y * b.y, w.x * b.y - w.y * b.x}; }   // conj(w) b
__device__ __forceinline__ cf mul_mi(cf a) { return {a.y, -a.x}; }   // -i a

// ------------------------------------------------------------------ small DFTs in registers

__device__ __forceinline__ void dft4(cf& a, cf& b, cf& c, cf& d) {
  const cf t0 = a + c, t1 = a - c, t2 = b + d, t3 = mul_mi(b - d);
  a = t0 + t2; b = t1 + t3; c = t0 - t2; d = t1 - t3;
}

template <int R>
__device__ __forceinline__ void dft(cf (&v)[R]) {
  if constexpr (R == 4) {
    dft4(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 8) {
    constexpr float h = 0.70710678118654752f;
    dft4(v[0], v[2], v[4], v[6]);
    dft4(v[1], v[3], v[5], v[7]);
    const cf o1 = {h * (v[3].x + v[3].y), h * (v[3].y - v[3].x)};      // W8 v
    const cf o2 = mul_mi(v[5]);
    const cf o3 = {h * (v[7].y - v[7].x), -h * (v[7].x + v[7].y)};     // W8^3 v
    const cf e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
    v[0] = e0 + o0; v[4] = e0 - o0;
    v[1] = e1 + o1; v[5] = e1 - o1;
    v[2] = e2 + o2; v[6] = e2 - o2;
    v[3] = e3 + o3; v[7] = e3 - o3;
  } else {
    static_assert(R == 16);
    constexpr float c1 = 0.92387953251128676f, s1 = 0.38268343236508977f, h = 0.70710678118654752f;
#pragma unroll
    for (int n = 0; n < 4; ++n) dft4(v[n], v[4 + n], v[8 + n], v[12 + n]);   // v[4 k1 + n2]
    // W16^(n2 k1)
    v[5] = cmul(v[5], {c1, -s1});  v[6] = cmul(v[6], {h, -h});    v[7] = cmul(v[7], {s1, -c1});
    v[9] = cmul(v[9], {h, -h});    v[10] = mul_mi(v[10]);         v[11] = cmul(v[11], {-h, -h});
    v[13] = cmul(v[13], {s1, -c1}); v[14] = cmul(v[14], {-h, -h}); v[15] = cmul(v[15], {-c1, s1});
#pragma unroll
    for (int k = 0; k < 4; ++k) dft4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);   // X[k1 + 4 k2]
    // transpose the 4 x 4 result into natural order
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = a + 1; b < 4; ++b) { const cf t = v[4 * a + b]; v[4 * a + b] = v[4 * b + a]; v[4 * b + a] = t; }
  }
}

// ------------------------------------------------------------------ FFT of N points by T lanes

template <int N> struct Plan;
template <> struct Plan<64>   { static constexpr int E = 4,  R0 = 4,  R1 = 4,  R2 = 4; };
template <> struct Plan<128>  { static constexpr int E = 8,  R0 = 8,  R1 = 4,  R2 = 4; };
template <> struct Plan<256>  { static constexpr int E = 8,  R0 = 8,  R1 = 8,  R2 = 4; };
template <> struct Plan<512>  { static constexpr int E = 8,  R0 = 8,  R1 = 8,  R2 = 8; };
template <> struct Plan<1024> { static constexpr int E = 16, R0 = 16, R1 = 8, R2 = 8; };
template <> struct Plan<2048> { static constexpr int E = 16, R0 = 16, R1 = 16, R2 = 8; };

template <int N> constexpr int lanes_of() { return N / Plan<N>::E; }
template <int N> constexpr int pairs_of() { return Plan<N>::E / 2; }
template <int N> constexpr int buf_of() { return N + N / 16; }     // a group's LDS buffer, complex
__device__ __forceinline__ constexpr int pad(int i) { return i + (i >> 4); }

// A lane's places.  Every index below is a base that depends on the lane plus a constant of the
// unrolled loop (pad(i + c) = pad(i) + pad(c) for the multiples c of 16 and the aligned i that occur
// here), so that a lane holds a few addresses and the accesses carry the rest as immediates.
template <int N>
struct Lane {
  static constexpr int T = lanes_of<N>(), E = Plan<N>::E;
  int t;
  int own, pair, mir;         // pad of t; of t + 1 (pair j = 0); of the last pair's mirror
  int even, odd;              // sample of point t; of point t + T (E - 1)
  __device__ __forceinline__ explicit Lane(int t_)
      : t(t_), own(pad(t_)), pair(pad(t_ + 1)), mir(pad(N / 2 + T - 1 - t_)), even(2 * t_), odd(2 * T - 1 - 2 * t_) {}
  // point or frequency t + T s in the buffer
  __device__ __forceinline__ int slot(int s) const { return own + pad(T * s); }
  // frequencies k = t + 1 + T j and N - k of pair j in the buffer
  __device__ __forceinline__ int k_at(int j) const { return pair + pad(T * j); }
  __device__ __forceinline__ int m_at(int j) const { return mir + pad(T * (E / 2 - 1 - j)); }
  __device__ __forceinline__ int k_of(int j) const { return t + 1 + T * j; }
  // the sample that point t + T s of the reordered row is: even samples, then odd ones backwards
  __device__ __forceinline__ int sample(int s) const { return s < E / 2 ? even + 2 * T * s : odd + 2 * T * (E - 1 - s); }
};

// Orders a group's LDS accesses before and after.  Inside one wavefront they execute in order and
// only the compiler has to be told that another lane's data is read; a group of two wavefronts
// (N = 2048) takes the workgroup's barrier, which every group reaches alike.
template <int N>
__device__ __forceinline__ void group_sync() {
  if constexpr (lanes_of<N>() > kWave) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Twiddles of the second and third stage, as the table holds them: W^{(q mod Ns) r}, W = e^{-2 pi i /
// (Ns R)}, of butterflies q = t + T a and r = 1 .. R - 1, one row of T lanes after the other (where
// Ns divides T every butterfly of a lane has the same ones: one a).
template <int N, int R, int Ns>
struct Twiddle {
  static constexpr int T = lanes_of<N>(), NB = Ns <= T ? 1 : Plan<N>::E / R, kRows = NB * (R - 1);
  cf w[kRows];
  __device__ __forceinline__ void load(int t, const cf* __restrict__ tab) {
#pragma unroll
    for (int i = 0; i < kRows; ++i) w[i] = (tab + i * T)[(unsigned)t];
  }
  __device__ __forceinline__ cf at(int a, int r) const { return w[(NB == 1 ? 0 : a) * (R - 1) + r - 1]; }
};
template <int N> using Twiddle1 = Twiddle<N, Plan<N>::R1, Plan<N>::R0>;
template <int N> using Twiddle2 = Twiddle<N, Plan<N>::R2, Plan<N>::R0 * Plan<N>::R1>;
template <int N> constexpr int tw_rows() { return Twiddle1<N>::kRows + Twiddle2<N>::kRows; }

// One radix-R stage of the E points in x (point t + T s in slot s), Ns the product of the radices
// before it: butterfly q takes points q + (N / R) r, turned by its twiddles.
template <int N, int R>
__device__ __forceinline__ void first_stage(cf (&x)[Plan<N>::E]) {
  constexpr int NB = Plan<N>::E / R;
#pragma unroll
  for (int a = 0; a < NB; ++a) {
    cf v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = x[a + NB * r];
    dft<R>(v);
#pragma unroll
    for (int r = 0; r < R; ++r) x[a + NB * r] = v[r];
  }
}
template <int N, int R, int Ns>
__device__ __forceinline__ void stage(cf (&x)[Plan<N>::E], const Twiddle<N, R, Ns>& w) {
  constexpr int NB = Plan<N>::E / R;
#pragma unroll
  for (int a = 0; a < NB; ++a) {
    cf v[R];
    v[0] = x[a];
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(x[a + NB * r], w.at(a, r));
    dft<R>(v);
#pragma unroll
    for (int r = 0; r < R; ++r) x[a + NB * r] = v[r];
  }
}

// the outputs of a stage to their places in the order of the next one
template <int N, int R, int Ns>
__device__ __forceinline__ void exchange(cf (&x)[Plan<N>::E], const Lane<N>& ln, cf* buf) {
  constexpr int E = Plan<N>::E, T = lanes_of<N>(), NB = E / R;
  static_assert(T % Ns == 0 && (Ns * R) % 16 == 0 || Ns == 1);
  const int o = pad((ln.t / Ns) * (Ns * R) + (ln.t & (Ns - 1)));
  group_sync<N>();                    // the buffer's earlier readers are done
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int r = 0; r < R; ++r) buf[o + pad(T * R * a) + pad(r * Ns)] = x[a + NB * r];
  group_sync<N>();
#pragma unroll
  for (int s = 0; s < E; ++s) x[s] = buf[ln.slot(s)];
}

// In place: point t + T s in slot s before, frequency t + T s in slot s after.  (The inverse runs on
// swapped real and imaginary parts.)  The twiddles are loaded a stage ahead, for their latency to
// pass behind it, and anew for every transform (the opaque offset): kept over a
// kernel's transforms they would take some 50 registers and with them half of its wavefronts.
template <int N>
__device__ __forceinline__ void fft(cf (&x)[Plan<N>::E], const Lane<N>& ln, cf* buf, const cf* __restrict__ tw) {
  using P = Plan<N>;
  int again = 0;
  asm volatile("" : "+s"(again));
  Twiddle1<N> w1;
  w1.load(ln.t, tw + again);
  first_stage<N, P::R0>(x);
  exchange<N, P::R0, 1>(x, ln, buf);
  asm volatile("" : "+s"(again));
  Twiddle2<N> w2;
  w2.load(ln.t, tw + again + Twiddle1<N>::kRows * lanes_of<N>());
  stage<N, P::R1, P::R0>(x, w1);
  exchange<N, P::R1, P::R0>(x, ln, buf);
  stage<N, P::R2, P::R0 * P::R1>(x, w2);
}

// natural order to and from the buffer
template <int N>
__device__ __forceinline__ void put(const cf (&x)[Plan<N>::E], const Lane<N>& ln, cf* buf) {
  group_sync<N>();
#pragma unroll
  for (int s = 0; s < Plan<N>::E; ++s) buf[ln.slot(s)] = x[s];
  group_sync<N>();
}
template <int N>
__device__ __forceinline__ void get(cf (&x)[Plan<N>::E], const Lane<N>& ln, const cf* buf) {
  group_sync<N>();
#pragma unroll
  for (int s = 0; s < Plan<N>::E; ++s) x[s] = buf[ln.slot(s)];
}

// The pairs (k, N - k) of a lane: k = t + 1 + T j, j < E / 2, from 1 to N / 2 over the group (the last
// is its own mirror); frequency 0 is left to lane 0.
// w_k of a lane's pairs, loaded together
template <int N>
struct PairW {
  cf w[pairs_of<N>()];
  __device__ __forceinline__ PairW(const cf* __restrict__ tab, int t) {
#pragma unroll
    for (int j = 0; j < pairs_of<N>(); ++j) w[j] = (tab + 1 + lanes_of<N>() * j)[(unsigned)t];
  }
};

// ((c_k - i c_m) / 2 of a cosine series, (om c_m - i ok c_k) / 2 of a sine series) from (c_k, c_m)
// given the halves wk = 1/2 or ok / 2 and wm = 1/2 or om / 2
__device__ __forceinline__ cf series(bool sine, float wk, float wm, float ck, float cm) {
  return sine ? cf{wm * cm, -wk * ck} : cf{wk * ck, -wm * cm};
}

// ------------------------------------------------------------------ kernels

struct FftTabs { const cf *tx, *wx, *ty, *wy; };   // the stages' twiddles and w_k, k <= N / 2, per axis

// Groups of lanes per workgroup of the x pass.  Sixteen rows y (eight groups) write the transposed
// rows in runs of 64 bytes and pay where the grid fills the chip several times over, eight rows split
// small grids better; at sides of 512 and up the line is kWideRows rows of all maps (eight rows and
// sixteen, Ex, Ey and Ez: 2048 x 2048 x 4 278 and 262 us, 1024 x 2048 x 4 112.5 and 110.4,
// 512 x 2048 x 4 62.1 and 61.6; 2048 x 1024 x 4 115.4 and 116.5, 1024 x 1024 x 4 56.2 and 56.7, 2048 x 512 x 4
// 65.7 and 70.0, 2048 x 64 x 2 22.6 and 28.2).  Shorter sides have groups of 16
// or 32 lanes and keep eight.
constexpr int kWideRows = 8192;
template <int N, int G> constexpr int x_threads() { return G * lanes_of<N>(); }

// The sum of v over a group's lanes, the same in all of them.  at: two floats of LDS for a group of two
// wavefronts (N = 2048), which every group of the workgroup then reaches alike.
template <int N>
__device__ __forceinline__ float group_sum(float v, int t, float* at) {
  constexpr int T = lanes_of<N>();
  for (int m = (T < kWave ? T : kWave) / 2; m > 0; m >>= 1) v += __shfl_xor(v, m);
  if constexpr (T > kWave) {
    if (t % kWave == 0) at[t / kWave] = v;
    __syncthreads();
    v = at[0] + at[1];
  }
  return v;
}

// the maps of a launch (of one problem, or of the layers of a multi-die one)
struct FftMapIn { const float* p[kMaxMany]; };
struct FftMapOut { float* p[kMaxMany]; };

// x forward: rows (z, y), two per FFT, to t[x frequency][z][y], with the x normalisation.
// The rows are transformed less the mean of the two, which goes to mean[z][y / 2] and which only the y
// transform of x frequency 0 sees again: the rounding of a transform is relative to what it sums, and an
// even density is mostly its mean, which the potential leaves out.  (A mean never makes what is
// summed larger, whatever the rows hold.  One value a layer, the mean of 64 of its bins, did where one of
// them held a peak: a bin of 1e4 over a density of 0.85 on 1024 x 1024 x 2, phi's error 4.1e-5, 2.3e-7 so.)
template <int N, int G>
__global__ __launch_bounds__((x_threads<N, G>())) void k_fft_x(FftMapIn maps, int ny, int nz, FftTabs tb, FftMapOut outs,
                                                              FftMapOut means) {
  const float* __restrict__ rho = maps.p[blockIdx.y];
  float* __restrict__ out = outs.p[blockIdx.y];
  constexpr int E = Plan<N>::E, T = lanes_of<N>(), RW = 2 * G;
  constexpr int kBuf = G * buf_of<N>() * 2, kTileF = N * (RW + 1);      // floats
  __shared__ __attribute__((aligned(16))) float L[kBuf > kTileF ? kBuf : kTileF];
  const int t = threadIdx.x & (T - 1), f = threadIdx.x / T;
  const int row0 = xcd_swizzle((int)blockIdx.x, (int)gridDim.x) * RW, z = row0 / ny, y0 = row0 - z * ny;
  const Lane<N> ln(t);
  cf* buf = reinterpret_cast<cf*>(L) + f * buf_of<N>();
  cf x[E];
  {
    const float* a = rho + (size_t)(row0 + 2 * f) * N;
    const float* b = a + N;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const int i = ln.sample(s);
      x[s] = {a[i], b[i]};
    }
    float sum = 0.f;
#pragma unroll
    for (int s = 0; s < E; ++s) sum += x[s].x + x[s].y;
    const float mean = group_sum<N>(sum, t, reinterpret_cast<float*>(buf)) * (0.5f / N);
#pragma unroll
    for (int s = 0; s < E; ++s) x[s] = {x[s].x - mean, x[s].y - mean};
    if (t == 0) means.p[blockIdx.y][row0 / 2 + f] = mean;
  }
  fft<N>(x, ln, buf, tb.tx);
  const PairW<N> pw(tb.wx, t);
  put<N>(x, ln, buf);
  // both rows' coefficients of every pair, then the tile [x frequency][row] in LDS
  cf zk[pairs_of<N>()], zm[pairs_of<N>()];
#pragma unroll
  for (int j = 0; j < pairs_of<N>(); ++j) {
    zk[j] = buf[ln.k_at(j)];
    zm[j] = buf[ln.m_at(j)];
  }
  const cf z0 = buf[0];
  constexpr float c = 1.f / N;        // 1/2 from the pair, 2/N (1/N at frequency 0) from the series
  __syncthreads();
#pragma unroll
  for (int j = 0; j < pairs_of<N>(); ++j) {
    const int k = ln.k_of(j);
    const cf wk = pw.w[j];
    const cf ua = cmul({zk[j].x + zm[j].x, zk[j].y - zm[j].y}, wk);
    const cf ub = cmul({zk[j].y + zm[j].y, zm[j].x - zk[j].x}, wk);
    L[k * (RW + 1) + 2 * f] = c * ua.x;
    L[k * (RW + 1) + 2 * f + 1] = c * ub.x;
    if (k != N - k) {
      L[(N - k) * (RW + 1) + 2 * f] = -c * ua.y;
      L[(N - k) * (RW + 1) + 2 * f + 1] = -c * ub.y;
    }
  }
  if (t == 0) {
    L[2 * f] = c * z0.x;
    L[2 * f + 1] = c * z0.y;
  }
  __syncthreads();
  // four consecutive y of one frequency per thread
  constexpr int Q = RW / 4;
  for (int i = threadIdx.x; i < N * Q; i += x_threads<N, G>()) {
    const int k = i / Q, q = i % Q;
    const float* s = L + k * (RW + 1) + 4 * q;
    *reinterpret_cast<float4*>(out + ((size_t)k * nz + z) * ny + y0 + 4 * q) = make_float4(s[0], s[1], s[2], s[3]);
  }
}

struct FftYArgs {
  FftMapIn mean;                 // [nz][N / 2] what the x pass took off the rows
  float px2, py, py2, pz2;       // (pi / length)^2, pi / d_y
  const float* zmat;
  FftMapIn t;                    // [nx][nz][N]
  FftMapOut vg, vh;              // [nx / 2][N][nz][2], either may be null
};

// 1 / w2 to half an ulp: the hardware reciprocal and one Newton step
__device__ __forceinline__ float recip(float w2) {
  const float r = __builtin_amdgcn_rcpf(w2);
  return fmaf(fmaf(-w2, r, 1.f), r, r);
}

// pairs of x frequencies per workgroup (NZ groups of lanes each), at least a wavefront of threads
template <int N, int NZ> constexpr int y_pairs() { return NZ * lanes_of<N>() >= kWave ? 1 : kWave / (NZ * lanes_of<N>()); }
template <int N, int NZ> constexpr int y_threads() { return y_pairs<N, NZ>() * NZ * lanes_of<N>(); }

// y forward, z mixing, 1 / |omega|^2, y inverse, two x frequencies at a time.
// The NZ groups of a pair (kx, kx + 1) first take one FFT each: two layers of one of the two
// frequencies.  Then each makes the coefficients of its share of the (k, N - k) pairs, all layers.
// Then group i takes z frequency i: its FFTs hold kx and kx + 1 as the two rows, whose sizes are
// alike (two z frequencies of one kx are not: l = 0 can be 10^4 times the others, and a transform's
// rounding, relative to the larger, would swamp them), cosine and sine one after the other.
template <int N, int NZ>
__global__ __launch_bounds__((y_threads<N, NZ>()), 2) void k_fft_y(FftYArgs g, FftTabs tb) {
  constexpr int E = Plan<N>::E, T = lanes_of<N>(), NP = pairs_of<N>(), H = NZ / 2, NQ = NP / H, B = buf_of<N>();
  __shared__ __attribute__((aligned(16))) cf L[y_pairs<N, NZ>() * NZ * B];
  const int tid = threadIdx.x, t = tid & (T - 1), f = tid / T, i = f % NZ, pr = f / NZ, c = i / H, r = i % H;
  const int kx2 = xcd_swizzle((int)blockIdx.x, (int)gridDim.x) * y_pairs<N, NZ>() + pr, kx = 2 * kx2 + c;
  const Lane<N> ln(t);
  cf* buf = L + f * B;
  {
    cf x[E];
    const float* r0 = g.t.p[blockIdx.y] + ((size_t)kx * NZ + 2 * r) * N;
    const float* r1 = r0 + N;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const int n = ln.sample(s);
      x[s] = {r0[n], r1[n]};
    }
    // x frequency 0 gets the rows' means back, less the layer's, which goes to frequency (0, 0)
    float ref0 = 0.f, ref1 = 0.f;
    if (kx2 == pr) {                                     // its workgroup
      const float* m0 = g.mean.p[blockIdx.y] + (size_t)(2 * r) * (N / 2);
      float a[E], b[E];
#pragma unroll
      for (int s = 0; s < E; ++s) {
        const int n = ln.sample(s) / 2;
        a[s] = m0[n];
        b[s] = m0[N / 2 + n];
        ref0 += a[s];
        ref1 += b[s];
      }
      ref0 = group_sum<N>(ref0, t, reinterpret_cast<float*>(buf)) * (1.f / N);
      ref1 = group_sum<N>(ref1, t, reinterpret_cast<float*>(buf) + 2) * (1.f / N);
      if (kx == 0) {
#pragma unroll
        for (int s = 0; s < E; ++s) x[s] = {x[s].x + (a[s] - ref0), x[s].y + (b[s] - ref1)};
      } else {
        ref0 = ref1 = 0.f;
      }
    }
    fft<N>(x, ln, buf, tb.ty);
    if (t == 0) x[0] = {x[0].x + (float)N * ref0, x[0].y + (float)N * ref1};
    put<N>(x, ln, buf);
  }
  __syncthreads();
  // b[j][l] = (b_k, -b_m) of z frequency l for the group's share of the pairs, with the 1/2 of the
  // inverse; b0[l] at frequency 0 (the first share's lane 0)
  cf b[NQ][NZ], wq[NQ];
  float b0[NZ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) wq[j] = (tb.wy + 1 + T * j)[(unsigned)(t + T * NQ * r)];
  const float fx = (float)kx, wx2 = g.px2 * (fx * fx);
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int l = 0; l < NZ; ++l) b[j][l] = {0.f, 0.f};
#pragma unroll
  for (int l = 0; l < NZ; ++l) b0[l] = 0.f;
#pragma unroll
  for (int p = 0; p < H; ++p) {
    const cf* zb = L + (f - r + p) * B;
    const cf *zk_at = zb + ln.pair + pad(T * NQ) * r, *zm_at = zb + ln.mir + pad(T * NQ) * (H - 1 - r);
    float f0[NZ], f1[NZ];
#pragma unroll
    for (int l = 0; l < NZ; ++l) {
      f0[l] = g.zmat[2 * p * kMaxNz + l] * (1.f / N);          // 1/2 from the pair, 2/N from the series
      f1[l] = g.zmat[(2 * p + 1) * kMaxNz + l] * (1.f / N);
    }
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const cf zk = zk_at[pad(T * j)], zm = zm_at[pad(T * (NQ - 1 - j))];
      const cf va = {zk.x + zm.x, zk.y - zm.y}, vb = {zk.y + zm.y, zm.x - zk.x};
#pragma unroll
      for (int l = 0; l < NZ; ++l)
        b[j][l] = {fmaf(f1[l], vb.x, fmaf(f0[l], va.x, b[j][l].x)), fmaf(f1[l], vb.y, fmaf(f0[l], va.y, b[j][l].y))};
    }
    const cf z0 = zb[0];
#pragma unroll
    for (int l = 0; l < NZ; ++l) b0[l] = fmaf(f1[l], z0.y, fmaf(f0[l], z0.x, b0[l]));
  }
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int k = t + 1 + T * (r * NQ + j);
    const cf wk = wq[j];
    const float fk = (float)k, fm = (float)(N - k);
#pragma unroll
    for (int l = 0; l < NZ; ++l) {
      const cf u = cmul(b[j][l], wk);
      const float w2 = wx2 + g.pz2 * (float)(l * l);
      b[j][l] = {u.x * (0.5f * recip(fmaf(g.py2, fk * fk, w2))), u.y * (0.5f * recip(fmaf(g.py2, fm * fm, w2)))};
    }
  }
  __syncthreads();
  // to the groups of their z frequencies: [z frequency][kx parity][pair], in the pair's NZ buffers
  cf* share = L + pr * NZ * B;
#pragma unroll
  for (int l = 0; l < NZ; ++l) {
#pragma unroll
    for (int j = 0; j < NQ; ++j) share[l * B + c * (N / 2) + (r * NQ + j) * T + t] = b[j][l];
    if (r == 0 && t == 0) {
      const float w2 = wx2 + g.pz2 * (float)(l * l);
      share[l * B + N + c] = {w2 > 0.f ? b0[l] * recip(w2) : 0.f, 0.f};     // the (0, 0, 0) mode is dropped
    }
  }
  __syncthreads();
  cf q0[NP], q1[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    q0[j] = buf[j * T + t];
    q1[j] = buf[N / 2 + j * T + t];
  }
  // kx + 1 is brought near kx by a power of two (on a 1:48 die kx = 0 holds a thousand times kx = 1):
  // by the ratio of their |omega|^2 at the lowest y frequency, its root for the sine series, whose
  // coefficients carry one omega_y
  const float base = fmaf(g.pz2, (float)(i * i), g.py2), fe = (float)(2 * kx2), fo = fe + 1.f;
  const unsigned ratio = __float_as_uint(fmaf(g.px2, fo * fo, base) * recip(fmaf(g.px2, fe * fe, base))) >> 23;
  const float d0 = buf[N].x, d1 = buf[N + 1].x;
#pragma unroll 1
  for (int sine = 0; sine < 2; ++sine) {
    float* v = sine ? g.vh.p[blockIdx.y] : g.vg.p[blockIdx.y];
    if (!v) continue;
    // rows kx and kx + 1 as g0 + i g1, real and imaginary parts swapped (an inverse FFT)
    const PairW<N> pw(tb.wy, t);
    const int e = min((int)ratio - 127, 96), up = sine ? e >> 1 : e;
    const float grow = __uint_as_float((unsigned)(127 + up) << 23), shrink = __uint_as_float((unsigned)(127 - up) << 23);
    group_sync<N>();
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const int k = ln.k_of(j);
      const float ok = sine ? g.py * (float)k : 1.f, om = sine ? g.py * (float)(N - k) : 1.f;
      const cf g0 = conj_mul(pw.w[j], series(sine, ok, om, q0[j].x, -q0[j].y));
      const cf g1 = conj_mul(pw.w[j], series(sine, grow * ok, grow * om, q1[j].x, -q1[j].y));
      buf[ln.m_at(j)] = {g1.x - g0.y, g0.x + g1.y};      // conj g0 + i conj g1
      buf[ln.k_at(j)] = {g0.y + g1.x, g0.x - g1.y};      // g0 + i g1
    }
    if (t == 0) buf[0] = sine ? cf{0.f, 0.f} : cf{grow * d1, d0};
    cf x[E];
    get<N>(x, ln, buf);
    fft<N>(x, ln, buf, tb.ty);
    // samples in y order, (kx, kx + 1) of this z frequency in its group's buffer; then every z
    // frequency of a sample as one run
    group_sync<N>();
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const bool neg = sine && s >= E / 2;               // odd samples of a sine series
      buf[ln.sample(s)] = {neg ? -x[s].y : x[s].y, (neg ? -shrink : shrink) * x[s].x};
    }
    __syncthreads();
    float* o = v + (size_t)kx2 * N * (2 * NZ);
    for (int u = (int)(tid % (NZ * T)); u < N * H; u += NZ * T) {
      const int y = u / H, l = 2 * (u % H);
      const cf e0 = share[l * B + y], e1 = share[(l + 1) * B + y];
      *reinterpret_cast<f32x4*>(o + 4 * u) = (f32x4){e0.x, e0.y, e1.x, e1.y};
    }
    __syncthreads();
  }
}

// one output map of the x inverse: its inverse-y source, z matrix, x series and destination
struct FftXJob { const float* v; const float* zm; int sine; float* out; };
struct FftXArgs { int ny; float px; int vec; FftXJob job[4 * kMaxMany]; };

// z mixing and x inverse of a few rows y of a map (blockIdx.y), one group of lanes each, two layers
// per FFT.  The rows' coefficients are read as the y pass wrote them, one run of 128 bytes (NZ = 4)
// for a pair of frequencies of four rows, and turned to rows in LDS, two z frequencies at a time.
// Two rows where four would leave one workgroup to a compute unit's registers (2048 x 2048 x 4, all
// four maps: 180 -> 153 us) or few to the chip (512 x 512 x 4, E: 9.3 -> 8.5); at 1024 four are as good.
template <int N> constexpr int ix_rows() { return N == 512 || N == 2048 ? 2 : 4; }
template <int N> constexpr int ix_threads() { return ix_rows<N>() * lanes_of<N>(); }

template <int N, int NZ>
__global__ __launch_bounds__(ix_threads<N>(), (N == 2048 ? 2 : 3)) void k_fft_ix(FftXArgs g, FftTabs tb) {
  constexpr int E = Plan<N>::E, T = lanes_of<N>(), NP = pairs_of<N>(), H = NZ / 2, RW = ix_rows<N>();
  constexpr int S = N + 16, kBuf = 2 * RW * buf_of<N>(), kStage = 2 * RW * S;     // floats
  __shared__ __attribute__((aligned(16))) float L[kBuf > kStage ? kBuf : kStage];
  const FftXJob J = g.job[blockIdx.y];
  const int tid = threadIdx.x, t = tid & (T - 1), f = tid / T, ny = g.ny;
  const int y0 = xcd_swizzle((int)blockIdx.x, (int)gridDim.x) * RW, y = y0 + f;
  const Lane<N> ln(t);
  cf* buf = reinterpret_cast<cf*>(L) + f * buf_of<N>();
  f32x4 in[E / 2][H];
  {
    const float* at = J.v + (size_t)(y0 + (tid & (RW - 1))) * (2 * NZ);
#pragma unroll
    for (int e = 0; e < E / 2; ++e)
#pragma unroll
      for (int h = 0; h < H; ++h)
        in[e][h] = *reinterpret_cast<const f32x4*>(at + (size_t)((tid / RW) + T * e) * ny * (2 * NZ) + 4 * h);
  }
  // (c_k, c_m) of every pair and layer, and c_0
  cf c[NZ][NP];
  float c0[NZ];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (h > 0) __syncthreads();
    float* at = L + (tid & (RW - 1)) * S + 2 * (tid / RW);
#pragma unroll
    for (int e = 0; e < E / 2; ++e) {
      *reinterpret_cast<f32x2*>(at + 2 * T * e) = (f32x2){in[e][h][0], in[e][h][1]};
      *reinterpret_cast<f32x2*>(at + RW * S + 2 * T * e) = (f32x2){in[e][h][2], in[e][h][3]};
    }
    __syncthreads();
#pragma unroll
    for (int l = 2 * h; l < 2 * h + 2; ++l) {
      const float* row = L + ((l & 1) * RW + f) * S;
      const float v0 = row[0];
#pragma unroll
      for (int z = 0; z < NZ; ++z) c0[z] = l == 0 ? J.zm[z] * v0 : fmaf(J.zm[l * kMaxNz + z], v0, c0[z]);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const float vk = (row + 1 + T * j)[t], vm = (row + N / 2 + T * (NP - 1 - j))[T - 1 - t];
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
          const float m = J.zm[l * kMaxNz + z];
          c[z][j] = l == 0 ? cf{m * vk, m * vm} : cf{fmaf(m, vk, c[z][j].x), fmaf(m, vm, c[z][j].y)};
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // this z frequency's values are used up before the next one's are read
    }
  }
  __syncthreads();
  const bool sine = J.sine != 0;
  const float hpx = 0.5f * g.px;
#pragma unroll
  for (int p = 0; p < NZ / 2; ++p) {
    const PairW<N> pw(tb.wx, t);
    group_sync<N>();
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const int k = ln.k_of(j);
      const cf a = c[2 * p][j], b = c[2 * p + 1][j];
      const float ok = sine ? hpx * (float)k : 0.5f, om = sine ? hpx * (float)(N - k) : 0.5f;
      const cf g0 = conj_mul(pw.w[j], series(sine, ok, om, a.x, a.y));
      const cf g1 = conj_mul(pw.w[j], series(sine, ok, om, b.x, b.y));
      buf[ln.m_at(j)] = {g1.x - g0.y, g0.x + g1.y};
      buf[ln.k_at(j)] = {g0.y + g1.x, g0.x - g1.y};
    }
    if (t == 0) buf[0] = sine ? cf{0.f, 0.f} : cf{c0[2 * p + 1], c0[2 * p]};
    cf x[E];
    get<N>(x, ln, buf);
    fft<N>(x, ln, buf, tb.tx);
    group_sync<N>();
    float* rows = reinterpret_cast<float*>(buf);
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const int i = ln.sample(s);
      const bool neg = sine && s >= E / 2;
      rows[i] = neg ? -x[s].y : x[s].y;
      rows[N + i] = neg ? -x[s].x : x[s].x;
    }
    group_sync<N>();
    float* o0 = J.out + ((size_t)(2 * p) * ny + y) * N;
    float* o1 = o0 + (size_t)ny * N;
    if (g.vec) {
#pragma unroll
      for (int s = 0; s < E / 4; ++s) {
        const int i = 4 * (t + T * s);
        *reinterpret_cast<float4*>(o0 + i) = *reinterpret_cast<const float4*>(rows + i);
        *reinterpret_cast<float4*>(o1 + i) = *reinterpret_cast<const float4*>(rows + N + i);
      }
    } else {
#pragma unroll
      for (int s = 0; s < E; ++s) {
        const int i = t + T * s;
        o0[i] = rows[i];
        o1[i] = rows[N + i];
      }
    }
  }
}

// the stages' twiddles (rows of T lanes, as Twiddle reads them) and w_k = e^{-i pi k / 2N}, k <= N / 2
template <int N>
__global__ void k_fft_tables(cf* __restrict__ tw, cf* __restrict__ wk) {
  constexpr int T = lanes_of<N>(), n1 = Twiddle1<N>::kRows, R1 = Plan<N>::R1, R2 = Plan<N>::R2, R0 = Plan<N>::R0;
  const int i = blockIdx.x * blockDim.x + threadIdx.x, row = i / T, t = i % T;
  if (row < tw_rows<N>()) {
    const int q = row < n1 ? row : row - n1, R = row < n1 ? R1 : R2, Ns = row < n1 ? R0 : R0 * R1;
    const int a = q / (R - 1), r = q % (R - 1) + 1;
    const double w = 2.0 * M_PI * (((t + T * a) % Ns) * r) / (Ns * R);
    tw[i] = {(float)cos(w), (float)-sin(w)};
  }
  if (i <= N / 2) {
    const double w = M_PI * i / (2.0 * N);
    wk[i] = {(float)cos(w), (float)-sin(w)};
  }
}

FftTabs tabs_of(const place3d_ctx* c) {
  auto p = [](const float2* q) { return reinterpret_cast<const cf*>(q); };
  return {p(c->fft.tx), p(c->fft.wx), p(c->fft.ty), p(c->fft.wy)};
}

// calls f with the compile-time side
template <class F>
void with_side(int n, F f) {
  switch (n) {
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    case 256: f(std::integral_constant<int, 256>{}); break;
    case 512: f(std::integral_constant<int, 512>{}); break;
    case 1024: f(std::integral_constant<int, 1024>{}); break;
    default: f(std::integral_constant<int, 2048>{}); break;
  }
}

}  // namespace

int build_fft(place3d_ctx* c, hipStream_t s) {
  if (!c->fft.on) return PLACE3D_OK;
  auto tables = [&](int n, float2* tw, float2* wk) {
    with_side(n, [&](auto side) {
      constexpr int N = decltype(side)::value;
      static_assert(tw_rows<N>() * lanes_of<N>() <= kFftTable * N && N / 2 + 1 <= kFftTable * N);
      hipLaunchKernelGGL((k_fft_tables<N>), dim3(blocks_for(kFftTable * N, 256)), dim3(256), 0, s,
                         reinterpret_cast<cf*>(tw), reinterpret_cast<cf*>(wk));
    });
  };
  tables(c->g.nx, c->fft.tx, c->fft.wx);
  tables(c->g.ny, c->fft.ty, c->fft.wy);
  P3D_LAUNCH(c, "k_fft_tables");
  return PLACE3D_OK;
}

int field_fft(place3d_ctx* c, const float* rho, float* phi, float* ex, float* ey, float* ez, hipStream_t s) {
  return field_fft_many(&c, &rho, &phi, &ex, &ey, &ez, 1, s);
}

int field_fft_many(place3d_ctx* const* c, const float* const* rho, float* const* phi, float* const* ex, float* const* ey,
                   float* const* ez, int nb, hipStream_t s) {
  const Geom& g = c[0]->g;
  const place3d_problem& p = c[0]->prob;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const FftTabs tb = tabs_of(c[0]);
  const double dz = p.nz * 0.5 * (p.die_x / p.nx + p.die_y / p.ny);
  const double px = M_PI / p.die_x, py = M_PI / p.die_y, pz = M_PI / dz;
  ProfScope prof_(c[0], PLACE3D_STAGE_GEMM, s);
  prof_.launches = 3;
  // every context asks for the same outputs
  const bool need_g = phi[0] || ex[0] || ez[0], need_h = ey[0] != nullptr;
  FftMapIn in{}, t_in{}, mean_in{};
  FftMapOut t_out{}, mean_out{}, vg{}, vh{};
  for (int i = 0; i < nb; ++i) {
    in.p[i] = rho[i];
    t_in.p[i] = t_out.p[i] = c[i]->map_t;
    mean_in.p[i] = mean_out.p[i] = c[i]->fft.mean;
    vg.p[i] = need_g ? c[i]->map_vg : nullptr;
    vh.p[i] = need_h ? c[i]->map_vh : nullptr;
  }
  with_side(nx, [&](auto side) {
    constexpr int N = decltype(side)::value;
    auto go = [&](auto groups) {
      constexpr int G = decltype(groups)::value;
      hipLaunchKernelGGL((k_fft_x<N, G>), dim3(nz * ny / (2 * G), nb), dim3(x_threads<N, G>()), 0, s, in, ny, nz, tb,
                         t_out, mean_out);
    };
    if constexpr (N >= 512) {
      if (nb * nz * ny < kWideRows) return go(std::integral_constant<int, 4>{});
    }
    go(std::integral_constant<int, 8>{});
  });
  P3D_LAUNCH(c[0], "k_fft_x");
  if (!need_g && !need_h) return PLACE3D_OK;
  const FftYArgs ya{mean_in, (float)(px * px), (float)py, (float)(py * py), (float)(pz * pz), c[0]->dct.zmat, t_in, vg, vh};
  with_side(ny, [&](auto side) {
    constexpr int N = decltype(side)::value;
    const int pairs = nx / 2;
    if (nz == 2) hipLaunchKernelGGL((k_fft_y<N, 2>), dim3(pairs / y_pairs<N, 2>(), nb), dim3(y_threads<N, 2>()), 0, s, ya, tb);
    else hipLaunchKernelGGL((k_fft_y<N, 4>), dim3(pairs / y_pairs<N, 4>(), nb), dim3(y_threads<N, 4>()), 0, s, ya, tb);
  });
  P3D_LAUNCH(c[0], "k_fft_y");
  const float* Gz = c[0]->dct.zmat + kMaxNz * kMaxNz;
  const float* Hz = c[0]->dct.zmat + 2 * kMaxNz * kMaxNz;
  FftXArgs xa{};
  xa.ny = ny; xa.px = (float)px;
  int nj = 0;
  for (int i = 0; i < nb; ++i) {
    if (ex[i]) xa.job[nj++] = {vg.p[i], Gz, 1, ex[i]};
    if (ez[i]) xa.job[nj++] = {vg.p[i], Hz, 0, ez[i]};
    if (phi[i]) xa.job[nj++] = {vg.p[i], Gz, 0, phi[i]};
    if (ey[i]) xa.job[nj++] = {vh.p[i], Gz, 0, ey[i]};
  }
  uintptr_t at = 0;
  for (int i = 0; i < nj; ++i) at |= reinterpret_cast<uintptr_t>(xa.job[i].out);
  xa.vec = (at & 15) == 0;
  with_side(nx, [&](auto side) {
    constexpr int N = decltype(side)::value;
    const dim3 grid(ny / ix_rows<N>(), nj);
    if (nz == 2) hipLaunchKernelGGL((k_fft_ix<N, 2>), grid, dim3(ix_threads<N>()), 0, s, xa, tb);
    else hipLaunchKernelGGL((k_fft_ix<N, 4>), grid, dim3(ix_threads<N>()), 0, s, xa, tb);
  });
  P3D_LAUNCH(c[0], "k_fft_ix");
  return PLACE3D_OK;
}

}  // namespace p3d
