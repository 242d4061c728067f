// bf_weights.hip -- weight generation on the device (FP64) and the MFMA
// operand layout of the weights.
//
// Phase model of Eq. 1 (Sec. 1): steering beam b to the unit direction k_b
// applies to antenna n at r_n the phase shift
//     W[c][b][n] = exp(-i 2 pi f_c (k_b . r_n) / c0).
// Sec. 3.2 recomputes coefficients whenever pointings change, overlapped
// with the previous iteration; here that is one kernel per bf_set_weights.
//
// Numerics: the phase in cycles f (k.r)/c0 reaches ~10^3 for a 500 m array
// at 416 MHz, so it is formed in FP64, reduced to [-1/2, 1/2] cycles in
// FP64 (exact subtraction of the nearest integer), and only then passed to
// sine and cosine (FP64).  Each weight component is rounded once, to nearest even,
// directly from FP64 to the storage format (no FP64 -> FP32 -> FP16 double
// rounding).
//
// Operand layout (what the beamform kernel stages in LDS):
//     w[c][bp][h][k],  bp < Bpad (B rounded up to 16), h = 0 (re-row) or
//     1 (im-row), k < Kpad (2N rounded up to 64);
//     re-row: k = 2n -> Re W, k = 2n+1 -> -Im W
//     im-row: k = 2n -> Im W, k = 2n+1 ->  Re W
// and zero for b >= B or n >= N, so that Re(W x) = re-row . [xr, xi] and
// Im(W x) = im-row . [xr, xi] over interleaved voltages.
#include "bf_internal.h"

namespace bf {

constexpr double kC0 = 299792458.0;  // m/s

// FP64 -> FP32 rounded to odd: the value itself if FP32 holds it, else the
// neighbour (of the two around it) whose last mantissa bit is set.  Rounding
// that to nearest even in a format with at least two bits fewer gives the FP64
// value rounded once: the odd bit stands for everything below it.
__device__ __forceinline__ float to_odd(double d) {
  const float f = (float)d;
  const double e = d - (double)f;  // exact
  uint32_t u = __float_as_uint(f);
  if ((u & 1u) == 0u && (e < 0.0 || e > 0.0))  // an even neighbour was taken: step toward d
    u += ((e < 0.0) == (u >> 31 != 0u)) ? 1u : 0xFFFFFFFFu;
  return __uint_as_float(u);
}

// One component in the storage format.
template <int PREC>
__device__ __forceinline__ uint32_t round_to(double v) {
  if constexpr (PREC == 0) return __float_as_uint((float)v);  // IEEE RNE
  if constexpr (PREC == 1) return __builtin_bit_cast(uint16_t, (_Float16)to_odd(v));
  return __builtin_bit_cast(uint16_t, (__bf16)to_odd(v));
}

// Antenna n's entries (2n, 2n+1) of the re-row, [Re W, -Im W], and the
// im-row, [Im W, Re W], as one (FP16, BF16) or two (FP32) dwords each.  The
// sign of a rounded value is flipped, not the value rounded twice.
template <int PREC>
__device__ __forceinline__ void entries(double wr, double wi, uint32_t* re, uint32_t* im) {
  const uint32_t r = round_to<PREC>(wr), i = round_to<PREC>(wi);
  if constexpr (PREC == 0) {
    re[0] = r;
    re[1] = i ^ 0x80000000u;
    im[0] = i;
    im[1] = r;
  } else {
    re[0] = r | ((i ^ 0x8000u) << 16);
    im[0] = i | (r << 16);
  }
}

// sin and cos of 2 pi frac, |frac| <= 1/2.  The angle is split into quarter
// turns and a rest t of at most an eighth of a turn, t in half turns (exact),
// and both functions are summed from their Taylor series in pi t: terms up to
// (pi t)^17 / 17! and (pi t)^16 / 16!, the next ones below 2^-58.  Multiples of
// a quarter turn come out exact.
__device__ __forceinline__ void sincos_turns(double frac, double* sn, double* cs) {
  const double k = rint(4.0 * frac);
  const double t = __builtin_fma(-0.5, k, 2.0 * frac);
  const double z = t * t;
  double s = 7.952054001475513e-07, c = 4.303069587032947e-06;
  s = __builtin_fma(s, z, -2.1915353447830217e-05);
  c = __builtin_fma(c, z, -0.0001046381049248457);
  s = __builtin_fma(s, z, 0.00046630280576761255);
  c = __builtin_fma(c, z, 0.0019295743094039231);
  s = __builtin_fma(s, z, -0.0073704309457143504);
  c = __builtin_fma(c, z, -0.02580689139001406);
  s = __builtin_fma(s, z, 0.08214588661112823);
  c = __builtin_fma(c, z, 0.2353306303588932);
  s = __builtin_fma(s, z, -0.5992645293207921);
  c = __builtin_fma(c, z, -1.3352627688545895);
  s = __builtin_fma(s, z, 2.5501640398773455);
  c = __builtin_fma(c, z, 4.0587121264167685);
  s = __builtin_fma(s, z, -5.16771278004997);
  c = __builtin_fma(c, z, -4.934802200544679);
  s = __builtin_fma(s, z, 3.141592653589793) * t;
  c = __builtin_fma(c, z, 1.0);
  const int q = (int)k;  // quarter turns, -2 .. 2
  const double a = q & 1 ? c : s, b = q & 1 ? s : c;
  // q = 0: (s, c); 1: (c, -s); -1: (-c, s); 2, -2: (-s, -c); no negative zeros
  *sn = ((q & 2) != 0 ? -a : a) + 0.0;
  *cs = (((q + 1) & 2) != 0 ? -b : b) + 0.0;
}

// a / c0 rounded to nearest, from the correctly rounded reciprocal and one
// correction by the exact remainder.
__device__ __forceinline__ double over_c0(double a) {
  constexpr double inv = 1.0 / kC0;
  const double q = a * inv;
  return __builtin_fma(__builtin_fma(-q, kC0, a), inv, q);
}

constexpr int kAnt = 4;  // antennas per thread

// A thread owns kAnt consecutive antennas of one beam and walks `cpt`
// channels: the projections k.r are formed once, and each operand row gets one
// 16-byte store (two in FP32).  mask[n] == 0 drops antenna n (zero weight
// column: a sub-array beam); absent beams and antennas (padding) are written as
// zeros.
// What bounds it: FP64 and rounding arithmetic, then the stores.  Per weight
// 18 FP64 multiply-adds of sine and cosine, 12 around them and about 16
// instructions of rounding; one row per workgroup with the library's sincospi,
// a division and integer rounding of all three stored components took about
// 185.  Measured per bf_set_weights call (its upload included) at N = 256, 512
// beams, 256 channels: FP16 (268 MB of rows) 230 -> 124 us, FP32 141 -> 123 (the
// stores of 537 MB take 107).
template <int PREC>
__global__ void __launch_bounds__(256) weights_geom_kernel(
    const double* __restrict__ pos, const double* __restrict__ dir,
    const double* __restrict__ freq, const double* __restrict__ mask, int N, int C, int B,
    int Bpad, int Kpad, int cpt, uint32_t* __restrict__ w) {
  constexpr int kDw = PREC == 0 ? 2 : 1;  // dwords per antenna and row
  const int groups = Kpad / (2 * kAnt);   // antenna groups per row
  const int64_t item = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (item >= (int64_t)Bpad * groups) return;
  const int b = (int)(item / groups);
  const int n0 = (int)(item - (int64_t)b * groups) * kAnt;
  double kr[kAnt];
  bool live[kAnt];
#pragma unroll
  for (int a = 0; a < kAnt; ++a) {
    const int n = n0 + a;
    live[a] = n < N && b < B && mask[n] != 0.0;
    kr[a] = 0.0;
    if (live[a])
      kr[a] = dir[3 * b] * pos[3 * n] + dir[3 * b + 1] * pos[3 * n + 1] +
              dir[3 * b + 2] * pos[3 * n + 2];  // m
  }
  const int64_t step = (int64_t)gridDim.y * cpt;
  for (int64_t cb = (int64_t)blockIdx.y * cpt; cb < C; cb += step) {
    const int ce = (int)(cb + cpt < C ? cb + cpt : C);
    for (int c = (int)cb; c < ce; ++c) {
      const double f = freq[c];
      uint32_t re[kAnt * kDw], im[kAnt * kDw];
#pragma unroll
      for (int a = 0; a < kAnt; ++a) {
        const double cyc = over_c0(f * kr[a]);  // phase in cycles
        double sn, cs;
        sincos_turns(cyc - rint(cyc), &sn, &cs);  // the difference is exact
        // exp(-i phi) = cos(phi) - i sin(phi)
        entries<PREC>(live[a] ? cs : 0.0, live[a] ? -sn : 0.0, re + a * kDw, im + a * kDw);
      }
      uint32_t* row = w + (((int64_t)c * Bpad + b) * 2 * Kpad + 2 * n0) * kDw / 2;
      uint4* r4 = reinterpret_cast<uint4*>(row);
      uint4* i4 = reinterpret_cast<uint4*>(row + (int64_t)Kpad * kDw / 2);
#pragma unroll
      for (int v = 0; v < kDw; ++v) {
        r4[v] = uint4{re[4 * v], re[4 * v + 1], re[4 * v + 2], re[4 * v + 3]};
        i4[v] = uint4{im[4 * v], im[4 * v + 1], im[4 * v + 2], im[4 * v + 3]};
      }
    }
  }
}

// Raw complex weights [C][B][N][2] (device copy) -> operand layout.
template <int PREC>
__global__ void __launch_bounds__(64) weights_raw_kernel(const double* __restrict__ wraw, int N,
                                                         int C, int B, int Bpad, int Kpad,
                                                         void* w) {
  const int half = Kpad / 2;
  const int64_t rows = (int64_t)C * Bpad;
  for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
    const int b = (int)(row % Bpad);
    const int64_t c = row / Bpad;
    for (int n = threadIdx.x; n < half; n += blockDim.x) {
      double wr = 0.0, wi = 0.0;
      if (n < N && b < B) {
        const double* src = wraw + ((c * B + b) * N + n) * 2;
        wr = src[0];
        wi = src[1];
      }
      constexpr int kDw = PREC == 0 ? 2 : 1;
      uint32_t re[kDw], im[kDw];
      entries<PREC>(wr, wi, re, im);
      uint32_t* r0 = reinterpret_cast<uint32_t*>(w) + (row * 2 * Kpad + 2 * n) * kDw / 2;
#pragma unroll
      for (int v = 0; v < kDw; ++v) {
        r0[v] = re[v];
        r0[(int64_t)Kpad * kDw / 2 + v] = im[v];
      }
    }
  }
}

__global__ void queue_clear_kernel(int32_t* q, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) q[i] = 0;
}

// Copies a set table from the kernel arguments into device memory, one dword
// per thread per step.
__global__ void __launch_bounds__(kThreads) table_store_kernel(const Launch L, Launch* dst) {
  static_assert(sizeof(Launch) % 4 == 0, "the table is copied in dwords");
  const uint32_t* src = reinterpret_cast<const uint32_t*>(&L);
  uint32_t* d = reinterpret_cast<uint32_t*>(dst);
  for (int i = threadIdx.x; i < (int)(sizeof(Launch) / 4); i += kThreads) d[i] = src[i];
}

// One workgroup per operand row, at most 2^20 of them (each then loops).
static int grid_rows(int64_t rows) {
  return (int)(rows < (1 << 20) ? (rows > 0 ? rows : 1) : (1 << 20));
}

template <typename K, typename... A>
static hipError_t launch(K kern, int grid, int block, hipStream_t s, A... a) {
  void* args[] = {reinterpret_cast<void*>(&a)...};
  return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid), dim3(block), args, 0, s);
}

hipError_t launch_weights_geom(int prec, const double* pos, const double* dir, const double* freq,
                               const double* mask, int N, int C, int B, int Bpad, int Kpad,
                               void* w, hipStream_t s) {
  const int64_t items = (int64_t)Bpad * (Kpad / (2 * kAnt));
  // channels per thread: enough threads to fill the device come first (about
  // 2^19), then sharing the projections over up to 16 channels
  int64_t cpt = items * C >> 19;
  cpt = cpt < 1 ? 1 : cpt > 16 ? 16 : cpt;
  const int64_t ny = (C + cpt - 1) / cpt;
  const dim3 grid((unsigned)((items + 255) / 256), (unsigned)(ny < 65535 ? ny : 65535));
  int cp = (int)cpt;
  uint32_t* wd = static_cast<uint32_t*>(w);
  void* args[] = {&pos, &dir, &freq, &mask, &N, &C, &B, &Bpad, &Kpad, &cp, &wd};
  const void* k = prec == 0   ? reinterpret_cast<const void*>(weights_geom_kernel<0>)
                  : prec == 1 ? reinterpret_cast<const void*>(weights_geom_kernel<1>)
                              : reinterpret_cast<const void*>(weights_geom_kernel<2>);
  return hipLaunchKernel(k, grid, dim3(256), args, 0, s);
}

hipError_t launch_weights_raw(int prec, const double* wraw, int N, int C, int B, int Bpad,
                              int Kpad, void* w, hipStream_t s) {
  const int grid = grid_rows((int64_t)C * Bpad);
  if (prec == 0) return launch(weights_raw_kernel<0>, grid, 64, s, wraw, N, C, B, Bpad, Kpad, w);
  if (prec == 1) return launch(weights_raw_kernel<1>, grid, 64, s, wraw, N, C, B, Bpad, Kpad, w);
  return launch(weights_raw_kernel<2>, grid, 64, s, wraw, N, C, B, Bpad, Kpad, w);
}

hipError_t launch_queue_clear(int32_t* q, int n, hipStream_t s) {
  return launch(queue_clear_kernel, 1, 64, s, q, n);
}

hipError_t launch_table_store(const Launch& L, Launch* dst, hipStream_t s) {
  return launch(table_store_kernel, 1, kThreads, s, L, dst);
}

}  // namespace bf
