// bf_host.cpp -- host-side logic with no HIP dependency (see bf_host.h).
#include "bf_host.h"

#include <algorithm>
#include <cctype>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace bf {

namespace {

const Tile kVecTiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_VEC16
#undef BF_TILE
};
const Tile kMultiTiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_MULTI
#undef BF_TILE
};
const Tile kGenTiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_GENERIC
#undef BF_TILE
};
const Tile kIn4Tiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_IN4
#undef BF_TILE
};
const Tile kWideTiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_WIDE
#undef BF_TILE
};
const Tile kFastTiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_FAST
#undef BF_TILE
};
const Tile kStreamTiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_STREAM
#undef BF_TILE
};
const Tile kCxTiles[] = {
#define BF_TILE(MT, NBT, NBP, KRES) Tile{MT, NBT, NBP, KRES},
    BF_TILE_LIST_CX
#undef BF_TILE
};

template <size_t K>
std::vector<Tile> as_vector(const Tile (&a)[K]) {
  return std::vector<Tile>(a, a + K);
}

int gcd(int a, int b) { return b ? gcd(b, a % b) : a; }

int64_t floor_pow2(int64_t v) {
  int64_t r = 1;
  while (r <= v / 2) r *= 2;
  return r;
}

}  // namespace

int make_shape(int32_t N, int32_t C, int32_t B, int64_t T, int32_t I, int prec, uint32_t flags,
               int n_cu, Shape* out) {
  if (!out) return BF_ERR_INVALID_ARG;
  if (N < 1 || N > kMaxN || C < 1 || C > kMaxC || B < 1 || B > kMaxB || T < 1 || I < 1 ||
      T > kMaxT || T % I != 0)
    return BF_ERR_INVALID_ARG;
  if (prec != BF_FP32 && prec != BF_FP16 && prec != BF_BF16) return BF_ERR_INVALID_ARG;
  if (flags & ~(uint32_t)(BF_ACCUMULATE | BF_INPUT_4BIT | BF_OUTPUT_COMPLEX))
    return BF_ERR_INVALID_ARG;
  // complex beams are per sample and overwrite their output
  if ((flags & BF_OUTPUT_COMPLEX) && (I != 1 || (flags & BF_ACCUMULATE))) return BF_ERR_INVALID_ARG;
  // 4-bit rows are read 8 bytes (8 antennas) at a time
  if ((flags & BF_INPUT_4BIT) && N % 8 != 0) return BF_ERR_UNSUPPORTED;
  Shape s;
  s.N = N;
  s.C = C;
  s.B = B;
  s.T = T;
  s.I = I;
  s.prec = prec;
  s.flags = flags;
  s.in4 = (flags & BF_INPUT_4BIT) != 0;
  s.cx = (flags & BF_OUTPUT_COMPLEX) != 0;
  s.vec16 = (2 * N) % 16 == 0;
  s.Bpad = (B + 15) / 16 * 16;
  s.Kpad = (2 * N + kChunk - 1) / kChunk * kChunk;
  s.mode = s.cx ? kModeCx : mode_of(I);
  s.n_cu = n_cu > 0 ? n_cu : 256;
  *out = s;
  return BF_OK;
}

int es_of(int prec) { return prec == BF_FP32 ? 4 : 2; }

int mode_of(int32_t I) {
  return I == 1 ? kModeI1 : I == 2 ? kModeI2 : (I % 4 == 0 ? kModeGen4 : kModeGen);
}

size_t lds_bytes(int prec, int32_t Kpad, int nbt) {
  return (size_t)2 * 16 * (size_t)nbt * ((size_t)Kpad * (size_t)es_of(prec) + kLdsPad);
}

size_t split_lds_bytes(int prec, int32_t Kpad, int nbt) {
  const size_t row = (size_t)kChunk * (prec == BF_FP32 ? 6 : 2) + kLdsPad;  // per 64-wide chunk
  return (size_t)2 * 16 * (size_t)nbt * ((size_t)Kpad / kChunk) * row;
}

size_t tile_lds(int prec, int32_t Kpad, Tile t) {
  if (t.kres == -1) return 0;
  if (t.kres == 0 || t.kres > 1) return lds_bytes(prec, Kpad, t.nbt);
  return split_lds_bytes(prec, Kpad, t.nbt);
}

void schedule(int32_t I, int64_t T, int32_t* G, int32_t* QI, int32_t* SG) {
  const int64_t W = T / I;
  if (I == 1) {
    *G = 1;
    *QI = 1;
  } else if (I == 2) {
    *G = 2;
    *QI = 1;
  } else {
    *QI = (I + 3) / 4;
    *G = 4 * *QI;
  }
  *SG = (int32_t)((W + 15) / 16);
}

bool same_tile(const Tile& a, const Tile& b) {
  return a.mt == b.mt && a.nbt == b.nbt && a.nbp == b.nbp && a.kres == b.kres;
}

// Bytes of voltages one wave reaches over with v store groups: its own rows and
// those up to the last wave step's and store group's padding (I % 4 != 0: a
// step can reach into the store group behind the last one).
static int64_t wave_span(const Shape& s, int64_t v) {
  const int64_t rowb = s.in4 ? s.N : 2 * (int64_t)s.N;
  const int64_t pad = (s.mode == kModeGen ? 32 : 16) * (int64_t)s.I + 128;
  return (std::min(s.T, v * 16 * s.I) + pad) * rowb;
}
constexpr int64_t kSpanMax = 0x7FFFFF00;  // below the out-of-range marker 2^31

// sgw * (row tiles per store group) must be a multiple of MT
static int32_t base_sgw(const Shape& s, int32_t mt) {
  int32_t G, QI, SG;
  schedule(s.I, s.T, &G, &QI, &SG);
  return mt / gcd(mt, G);
}

bool buffer_shape(const Shape& s, int nbt) {
  const int64_t out = s.cx ? s.T : s.T / s.I;  // 4 bytes each
  return s.T < ((int64_t)1 << 31) && wave_span(s, base_sgw(s, 4)) < kSpanMax &&
         std::min((int64_t)s.B, (int64_t)16 * nbt) * out * 4 < kSpanMax;
}

int32_t wave_sgw(const Shape& s, const Tile& f, int32_t sgw) {
  if (f.kres == 0 || f.kres == -1 || wave_span(s, sgw) < kSpanMax) return sgw;
  const int64_t rowb = s.in4 ? s.N : 2 * (int64_t)s.N;
  const int32_t base = base_sgw(s, f.mt);
  const int64_t most = (kSpanMax - 1 - wave_span(s, 0)) / (16 * s.I * rowb);
  return (int32_t)std::max<int64_t>(base, most / base * base);
}

bool wide_shape(const Shape& s) {
  if (s.prec == BF_FP32 || s.cx || !s.vec16 || (s.flags & BF_ACCUMULATE)) return false;
  if (s.mode != kModeI1 && s.mode != kModeGen4) return false;
  // the whole channel and all its beams within one wave's reach
  return (s.T / s.I) % 4 == 0 && s.T < ((int64_t)1 << 31) && wave_span(s, s.T) < kSpanMax &&
         (int64_t)s.B * (s.T / s.I) * 4 < kSpanMax;
}

bool fast_ok(const Shape& s) {
  if (s.Kpad != kChunk || s.N % 2 != 0 || !buffer_shape(s, 1)) return false;
  if (s.mode == kModeGen4) return true;
  // I == 1 and complex beams: one beam tile, overwriting, whole 16-byte quads.
  // Wider ranges store tile by tile between MFMA phases here and are bound by
  // that write stream; the streamed form's bursts reach HBM better (N = 32,
  // 512 beams, I = 1, 4-bit BF16: 238 against 218 us).
  return (s.mode == kModeI1 || s.mode == kModeCx) && s.Bpad == 16 && s.T % 4 == 0 &&
         !(s.flags & BF_ACCUMULATE);
}

// The widest beam range the shape's beams fill beyond one of half the width
// and whose weights fit.  Four waves while two workgroups fit a CU (one
// stages its weights while the other computes), else eight.
bool stream_tile(const Shape& s, size_t lds_cap, Tile* t) {
  const int need = s.Bpad / 16;
  for (int nbt = 4; nbt >= 1; nbt /= 2) {
    if ((nbt > 1 && nbt / 2 >= need) || !buffer_shape(s, nbt)) continue;
    const size_t l = split_lds_bytes(s.prec, s.Kpad, nbt);
    if (l > lds_cap) continue;
    *t = Tile{4, nbt, nbt, l <= 80 * 1024 ? kKresStream4 : kKresStream8};
    return true;
  }
  return false;
}

Tile form_of(const Shape& s, Tile t) {
  if (t.kres == kKresWide) {
    // the name's own width, or the widest narrower one whose weights fit
    int nbt = t.nbt;
    while (nbt > 1 && split_lds_bytes(s.prec, s.Kpad, nbt) > kLdsMax) nbt /= 2;
    return Tile{4, nbt, nbt, kKresStream8};
  }
  if (t.kres >= 1) {
    if (t.kres == 1 && fast_ok(s) && buffer_shape(s, s.mode == kModeGen4 ? t.nbt : 1))
      return Tile{4, s.mode == kModeGen4 ? t.nbt : 1, 1, 1};
    Tile r;
    if (stream_tile(s, kLdsMax, &r)) return r;
    t.kres = 0;
  }
  if (t.kres != 0) return t;
  // general form: in 16 bits every beam tile of the range in one pass, at most
  // four; in FP32 two per pass (byte-load rows have no width of four there)
  if (t.nbt <= 2) return Tile{4, t.nbt, t.nbt, 0};
  if (s.prec != BF_FP32) return Tile{4, 4, 4, 0};
  return Tile{4, t.nbt == 8 || !s.vec16 ? 8 : 4, 2, 0};
}

std::vector<Tile> compiled_tiles(const Shape& s) {
  std::vector<Tile> v;
  if (s.cx && s.vec16)
    v = as_vector(kCxTiles);
  else if (s.in4)
    v = as_vector(kIn4Tiles);
  else if (s.vec16)
    v = as_vector(kVecTiles);
  else
    v = as_vector(kGenTiles);
  if (fast_ok(s))
    for (const Tile& t : kFastTiles) {
      bool named = (s.mode != kModeGen4 && t.nbt > 1) || !buffer_shape(s, t.nbt);
      for (const Tile& o : v) named = named || same_tile(o, t);
      if (!named) v.push_back(t);
    }
  if (wide_shape(s)) {
    v.push_back(Tile{4, 4, 4, kKresWide});
    v.push_back(Tile{4, 2, 2, kKresWide});
  }
  for (const Tile& t : kStreamTiles)
    // the eight-wave ranges that kres == -2 names are not offered twice
    if (buffer_shape(s, t.nbt) && !(t.kres == kKresStream8 && t.nbt > 1 && wide_shape(s)))
      v.push_back(t);
  return v;
}

std::vector<Tile> multi_tiles() { return as_vector(kMultiTiles); }

std::vector<Tile> wide_tiles() { return as_vector(kWideTiles); }

bool tile_exists(const Shape& s, Tile t) {
  for (const Tile& x : compiled_tiles(s))
    if (same_tile(x, t)) return true;
  return false;
}

bool tile_ok(const Shape& s, Tile t) {
  if (!tile_exists(s, t)) return false;
  if (t.kres > 0 && s.Kpad / kChunk > t.kres) return false;
  // names that an earlier form bounded by its own LDS rows
  if (t.kres == kKresWide && lds_bytes(s.prec, s.Kpad, t.nbt) > kLdsMax) return false;
  if (t.kres > 0 && lds_bytes(s.prec, s.Kpad, t.nbt) > kLdsMax) return false;
  return tile_lds(s.prec, s.Kpad, form_of(s, t)) <= kLdsMax;
}

std::vector<Tile> offered_tiles(const Shape& s) {
  std::vector<Tile> names, offered;
  for (const Tile& t : compiled_tiles(s))
    if (tile_ok(s, t)) names.push_back(t);
  for (size_t i = 0; i < names.size(); ++i) {
    const Tile f = form_of(s, names[i]);
    const bool own = same_tile(names[i], f);
    bool first = true;
    for (size_t j = 0; j < names.size() && first; ++j)
      if (j != i && same_tile(form_of(s, names[j]), f))
        first = own || (j > i && !same_tile(names[j], f));
    if (first) offered.push_back(names[i]);
  }
  return offered;
}

int64_t units_for(const Shape& s, Tile t, int32_t sgw) {
  const Tile f = form_of(s, t);
  int32_t G, QI, SG;
  schedule(s.I, s.T, &G, &QI, &SG);
  const int64_t nbr = (s.Bpad / 16 + f.nbt - 1) / f.nbt;
  const int64_t per = (int64_t)waves_of(f) * wave_sgw(s, f, sgw);
  const int64_t ntr = (SG + per - 1) / per;
  return (int64_t)s.C * nbr * ntr;
}

// Cycles of one unit of form f with v store groups per wave where wg of its
// workgroups share a CU, from a simple model: its weight staging (8000 cycles
// and 8 bytes a cycle) plus its wave steps.  A step costs the larger of two:
// its MFMA and VALU cycles (conversion per chunk, detection per beam tile),
// shared by the waves that are resident on the SIMD (one alone overlaps
// nothing: 1.4 times); and its HBM bytes at the CU's share of the bandwidth (8
// bytes a cycle; the voltages are fetched once for all beam ranges of a
// channel).
// The constants: 16 cycles per MFMA, 40 VALU instructions per row tile and half
// chunk of conversion and 32 of detection per beam and row tile are counted from
// the kernels; the others were set by hand.  Over 89 drawn single runs (N 2 to 512,
// B 1 to 1000, every precision, input and output), each timed under every form and
// unit length, the choice takes 1.07 of the best one's time on average (median
// 1.02, nine in ten below 1.18).  That mean is flat in the hand-set ones: staging 0
// or 16000 cycles 1.064, 1.069; 4 or 16 LDS bytes a cycle 1.069, 1.061; VALU weight
// 1 or 2.4 instead of 1.6 1.072, 1.056; the lone wave's 1.4 as 1 or 2 1.079, 1.065,
// and without its rule 1.085; 4 or 16 HBM bytes a cycle 1.089, 1.067.
double unit_cycles(const Shape& s, Tile f, int32_t v, int wg) {
  int32_t G, QI, SG;
  schedule(s.I, s.T, &G, &QI, &SG);
  const int nw = waves_of(f);
  const int need = s.Bpad / 16;
  const int nbr = (need + f.nbt - 1) / f.nbt;
  // the register-resident form computes every tile of its width
  const int bw = f.kres == 1 ? f.nbt : (need + nbr - 1) / nbr;
  const double groups = (double)(SG + v - 1) / v;  // waves with work in a channel's range
  const double waves = (double)wg * (groups < nw ? groups : nw);
  const double per_simd = waves > 5.6 ? waves / 4 : 1.4;
  const double parts = s.prec == BF_FP32 ? 3 : 1;
  const double halves = (2 * s.N + 31) / 32;
  const double rowb = s.in4 ? s.N : 2.0 * s.N;
  const double mfma = halves * bw * parts * f.mt * 2 * 16;
  const double valu = 1.6 * (halves * 40 * 4 + bw * 32.0 * f.mt);
  const double mem = waves * 16 * f.mt * (rowb / nbr + 64.0 * bw / s.I) / 8;
  const double work = (mfma + valu) * per_simd;
  const double step = work > mem ? work : mem;
  const double steps = s.mode == kModeGen ? s.I / 4.0 : (double)G / f.mt;  // per store group
  return 8000.0 + (double)tile_lds(s.prec, s.Kpad, f) / 8.0 + (v < SG ? v : SG) * steps * step;
}

// Cycles of one launch: units run over the device's workgroup slots in whole
// rounds, or, over many rounds, until a quarter of a unit after the last slot
// frees.  Eight waves cost 5% more at a tie.  (Over the same runs: half a unit or
// none instead of the quarter 1.066, 1.069; no 5% or 15% 1.062, 1.075.)
static double form_cycles(const Shape& s, const Tile& f, int32_t v) {
  int32_t G, QI, SG;
  schedule(s.I, s.T, &G, &QI, &SG);
  const int nw = waves_of(f);
  const int nbr = (s.Bpad / 16 + f.nbt - 1) / f.nbt;
  const size_t lds = tile_lds(s.prec, s.Kpad, f);
  // workgroups per CU by registers, then LDS
  int wg = nw == kWideWaves ? (f.nbt == 1 ? 2 : 1)
           : f.nbt == 1     ? 4
           : f.nbt == 2 && f.kres != 1 ? 3 : 2;
  while (wg > 1 && lds * wg > kLdsMax) --wg;
  const double units =
      (double)s.C * nbr * (double)((SG + (int64_t)nw * v - 1) / ((int64_t)nw * v));
  if (units < (double)s.n_cu * wg) wg = (int)std::ceil(units / s.n_cu);
  const double rounds = units / ((double)s.n_cu * wg);
  const double whole = std::ceil(rounds), tail = rounds + 0.25;
  return (whole > tail ? whole : tail) * unit_cycles(s, f, v, wg) *
         (nw == kWideWaves ? 1.05 : 1.0);
}

// The store groups per wave that finish first under form_cycles; *cycles: their
// cost.  Long units amortise the staging, short ones fill the device.  Against
// the counts that fill whole rounds: N = 32, 128 channels, B = 100, I = 5: 97.7
// -> 85 us.  Per-sample outputs (I == 1, complex) are bound by the write stream,
// which reaches HBM better in short runs: at most 16 groups, 4 for one beam tile
// (N = 32, 512 beams, I = 1: 218 us at 16, 222 at 32, 245 at 8; 16 complex
// beams: 762 at 4, 786 at 8, 816 at 32).  The general form at one chunk, which
// runs where rows are over 100 MB apart: 64 (N = 32, 64 beams, 35.6 M samples: 2.67
// to 2.86 ms at 16, 2.64 at 32 and 64, 2.78 at 256).  Over the runs of unit_cycles
// the mean is 1.066 with these caps, 1.068 with 64 for all.
static int32_t best_sgw(const Shape& s, const Tile& f, int32_t base, double* cycles) {
  int32_t G, QI, SG;
  schedule(s.I, s.T, &G, &QI, &SG);
  const int32_t most = s.I > 1 ? 1 << 20
                       : f.kres == 0 && s.Kpad == kChunk ? 64
                       : f.nbt == 1 ? 4 : 16;
  int32_t best = base;
  for (int32_t k = 1;; k = k < 4 ? k + 1 : k + k / 3) {
    if ((int64_t)base * k > most) break;
    const int32_t v = base * k;
    if (wave_sgw(s, f, v) != v) break;
    const double c = form_cycles(s, f, v);
    if (k == 1 || c < *cycles) {
      best = v;
      *cycles = c;
    }
    if ((int64_t)v * waves_of(f) >= SG) break;
  }
  return best;
}

int32_t choose_sgw(const Shape& s, Tile t) {
  double cycles = 0;
  return best_sgw(s, form_of(s, t), base_sgw(s, t.mt), &cycles);
}

// Default tile: the register-resident form (2N <= 64) or the streamed form (up
// to K = 2048) of the width and wave count that finish first under
// form_cycles.  Beyond, and for channels past 32-bit offsets, the general
// form: the largest beam range whose weight slice fits 80 KB of LDS (two
// workgroups per CU) without exceeding the plan's beams.
void choose_tile(const Shape& s, Tile* out, int32_t* out_sgw) {
  const int need = s.Bpad / 16;
  double least = 0;
  bool found = false;
  auto consider = [&](const Tile& t, const Tile& f) {
    if (tile_lds(s.prec, s.Kpad, f) > kLdsMax) return;
    if (f.nbt > 1 && f.kres != 1 && f.nbt / 2 >= need) return;
    double c = 0;
    const int32_t v = best_sgw(s, f, base_sgw(s, t.mt), &c);
    if (found && c >= least) return;
    found = true;
    least = c;
    *out = t;
    *out_sgw = v;
  };
  if (s.prec != BF_FP32 && s.vec16 && s.mode != kModeGen && need > 1 &&
      lds_bytes(s.prec, s.Kpad, 2) <= kLdsMax && split_lds_bytes(s.prec, s.Kpad, 2) > kLdsMax &&
      units_for(s, Tile{4, 2, 2, 0}, base_sgw(s, 4)) >= s.n_cu) {
    // N = 552 .. 608: two beam tiles' weights fit LDS only in the general form's
    // rows, which have no padding per chunk (N = 600 x 27 channels, 256 beams, 7680
    // samples, FP16, against the streamed form's one tile: I = 64 697 -> 465 us,
    // I = 16 653 -> 446, I = 1 147 -> 132; I = 5, with dummy rows, 602 -> 671).  With
    // fewer units than CUs one tile's twice as many finish first (N = 560 x 8
    // channels, 395 beams, 1344 4-bit samples, I = 64: 197 -> 136)
    *out = Tile{4, 2, 2, 0};
    *out_sgw = choose_sgw(s, *out);
    return;
  }
  // Where the output rows of the whole beam range do not fit the offsets (up to
  // four beam tiles; few samples per window, a channel past 2 GiB), narrower
  // ranges would read the voltages again for each: the register-resident form
  // takes the widest that fits (64 beams, FP16: N = 32 at I = 4 1.52 -> 1.29 ms, N = 8 at
  // I = 16 3.0, 4.7 in the general form), in 16 bits the general form's 64-bit rows
  // are faster than a narrower streamed one (N = 32 at I = 2 2.10 -> 1.49, N = 64 at I = 1
  // 1.91 -> 1.38; FP32 stays: N = 32 at I = 2 2.06 against 2.51).
  int range = 1, widest = 1;
  while (range < 4 && range < need) range *= 2;
  const bool narrow = !buffer_shape(s, range);
  for (const Tile& t : kFastTiles)
    if (t.nbt > widest && buffer_shape(s, t.nbt)) widest = t.nbt;
  if (fast_ok(s)) {
    for (const Tile& t : kFastTiles)
      if ((s.mode == kModeGen4 || t.nbt == 1) && t.nbt <= widest && (!narrow || t.nbt == widest))
        consider(t, t);
  } else if (narrow && s.prec != BF_FP32 && s.vec16 &&
             lds_bytes(s.prec, s.Kpad, range) <= 80 * 1024) {
    // the general form, below
  } else if (s.Kpad <= 2048) {
    for (const Tile& f : kStreamTiles) {
      Tile t = f;
      if (f.kres == kKresStream8 && f.nbt > 1 && wide_shape(s)) t.kres = kKresWide;
      if (tile_ok(s, t)) consider(t, f);
    }
  }
  if (found) return;
  Tile t{4, 1, 1, 0};
  const size_t lds1 = lds_bytes(s.prec, s.Kpad, 1);
  if (lds1 > kLdsMax ||
      (!s.vec16 && lds1 > 80 * 1024 && units_for(s, t, base_sgw(s, t.mt)) > s.n_cu)) {
    // one beam tile's weights do not fit LDS; or they leave one workgroup per
    // CU, whose four waves wait for each byte of a byte-load row (N = 1121 x 14
    // channels, 256 beams, FP16: I = 5 12.3 -> 4.6 ms, I = 64 9.6 -> 5.8, I = 1
    // 1.86 -> 0.89; 16 beams, I = 5: 1.13 -> 0.85; FP32, N = 601: 6.4 -> 2.5).
    // With no more units than CUs there is one per CU in either form, and LDS is
    // the faster (N = 1121 x 2 channels, 49984 samples, I = 64: 16 beams 4.91
    // against 4.67, 35 beams 5.15 against 4.66; FP32, N = 601: 3.02 against 2.79)
    t = Tile{4, 2, 2, -1};
  } else {
    int nbt = s.prec == BF_FP32 ? 8 : 4;
    while (nbt > 1 && (lds_bytes(s.prec, s.Kpad, nbt) > 80 * 1024 || nbt / 2 >= need)) nbt /= 2;
    if (!s.vec16) {
      // the byte-load rows' wide form, if the beams fill more than one tile
      const int wide = s.prec == BF_FP32 ? 8 : 4, least = s.prec == BF_FP32 ? 4 : 1;
      nbt = need > least && lds_bytes(s.prec, s.Kpad, wide) <= 80 * 1024 ? wide : 1;
    }
    t = nbt == 8 ? Tile{4, 8, 2, 0} : Tile{4, nbt, nbt, 0};
  }
  *out = t;
  *out_sgw = choose_sgw(s, t);
}

int multi_variant(const Shape& s, const Tile* own, size_t lds_cap) {
  const int n = (int)(sizeof(kMultiTiles) / sizeof(kMultiTiles[0]));
  auto runs = [&](const Tile& c, size_t cap) {
    if (tile_lds(s.prec, s.Kpad, c) > cap) return false;
    if (c.kres == 1) return s.mode == kModeGen4 && fast_ok(s) && buffer_shape(s, c.nbt);
    return c.kres == kKresStream4 ? buffer_shape(s, c.nbt) : true;
  };
  const Tile f = own ? form_of(s, *own) : Tile{0, 0, 0, 0};
  const int need = s.Bpad / 16;
  // two workgroups per CU if any variant allows it
  for (size_t cap : {lds_cap < 80 * 1024 ? lds_cap : (size_t)80 * 1024, lds_cap}) {
    for (int v = 0; v < n; ++v)
      if (same_tile(kMultiTiles[v], f) && runs(f, cap)) return v;
    for (int v = 0; v < n; ++v) {
      const Tile& c = kMultiTiles[v];
      if (c.nbt > 1 && c.nbt / 2 >= need) continue;  // half its width would do
      if (runs(c, cap)) return v;
    }
  }
  return -1;
}

int wide_variant(const Shape& s, size_t lds_cap, int32_t* sgw) {
  const int n = (int)(sizeof(kWideTiles) / sizeof(kWideTiles[0]));
  for (int v = 0; v < n; ++v) {
    const Tile& c = kWideTiles[v];
    if (!buffer_shape(s, c.nbt) || tile_lds(s.prec, s.Kpad, c) > lds_cap ||
        (c.nbt > 1 && s.Bpad / 16 <= c.nbt / 2))
      continue;
    int32_t G, QI, SG;
    schedule(s.I, s.T, &G, &QI, &SG);
    const int32_t base = c.mt / gcd(c.mt, G);
    *sgw = std::max(base, SG / kWideWaves / base * base);
    return v;
  }
  return -1;
}

bool wide_sets(const BatchSet* sets, int n, bool* wide) {
  int64_t want = 0, others = 0, cramped = 0;
  bool all = true;
  const int n_cu = n > 0 ? sets[0].s->n_cu : 256;
  for (int i = 0; i < n; ++i) {
    const Shape& s = *sets[i].s;
    wide[i] = form_of(s, sets[i].tile).kres == kKresStream8;
    (wide[i] ? want : others) += units_for(s, sets[i].tile, sets[i].sgw);
    int32_t sgw = 0;
    const int v = wide_variant(s, kLdsMax, &sgw);
    all = all && v >= 0 && s.Kpad > 2 * kChunk;
    if (v >= 0 && s.Bpad > 32 && split_lds_bytes(s.prec, s.Kpad, 4) > 80 * 1024)
      cramped += units_for(s, kWideTiles[v], sgw);
  }
  const bool cramp = sets[0].s->prec != BF_FP32 && sets[0].s->mode == kModeGen4 &&
                     4 * cramped >= 3 * (int64_t)n_cu;
  if (all && (want >= 2 * (int64_t)n_cu || cramp)) {
    for (int i = 0; i < n; ++i) wide[i] = true;
    return true;
  }
  return want >= 2 * (int64_t)n_cu && (others == 0 || others >= 4 * (int64_t)n_cu);
}

int check_tile(const Shape& s, Tile t, int32_t sgw) {
  if (sgw < 1) return BF_ERR_INVALID_ARG;
  if (!tile_ok(s, t)) return BF_ERR_UNSUPPORTED;
  int32_t G, QI, SG;
  schedule(s.I, s.T, &G, &QI, &SG);
  if (((int64_t)sgw * G) % t.mt != 0) return BF_ERR_INVALID_ARG;
  return BF_OK;
}

uint64_t input_bytes(const Shape& s) {
  const uint64_t row = s.in4 ? (uint64_t)s.N : 2 * (uint64_t)s.N;
  return (uint64_t)s.C * (uint64_t)s.T * row;
}

uint64_t output_bytes(const Shape& s) {
  const uint64_t per_beam = s.cx ? (uint64_t)s.T * 4 : (uint64_t)(s.T / s.I) * 4;
  return (uint64_t)s.C * (uint64_t)s.B * per_beam;
}

bool ranges_overlap(const void* a, uint64_t na, const void* b, uint64_t nb) {
  if (na == 0 || nb == 0) return false;
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  // [x, x + na) and [y, y + nb) intersect iff each starts before the other ends
  return x < y ? (y - x) < na : (x - y) < nb;
}

std::string tune_key(const Shape& s, bool batch, const char* arch) {
  char buf[256];
  std::snprintf(buf, sizeof(buf), "%s/p%d/N%d/B~%lld/I%d/C~%lld/T~%lld%s%s%s", arch ? arch : "",
                s.prec, s.N, (long long)floor_pow2(s.B), s.I, (long long)floor_pow2(s.C),
                (long long)floor_pow2(s.T), s.in4 ? "/in4" : "", s.cx ? "/cx" : "",
                batch ? "/batch" : "");
  return std::string(buf);
}

// ---- a minimal JSON reader for the tile cache ----
namespace {

class Reader {
 public:
  Reader(const char* p, size_t n) : p_(p), e_(p + n) {}

  // The whole text: one object whose members are cache entries.
  bool top(std::vector<TuneEntry>* out) {
    if (!lit('{')) return false;
    if (lit('}')) return end();
    for (;;) {
      std::string key;
      if (!str(&key) || !lit(':')) return false;
      TuneEntry e;
      bool good = false;
      if (peek() == '{') {
        if (!entry(&e, &good)) return false;
      } else if (!skip()) {
        return false;
      }
      if (good) {
        e.key = key;
        out->push_back(e);
      }
      if (lit(',')) continue;
      if (lit('}')) return end();
      return false;
    }
  }

 private:
  const char* p_;
  const char* e_;
  int depth_ = 0;

  void ws() {
    while (p_ < e_ && (*p_ == ' ' || *p_ == '\n' || *p_ == '\r' || *p_ == '\t')) ++p_;
  }
  char peek() {
    ws();
    return p_ < e_ ? *p_ : '\0';
  }
  bool lit(char c) {
    ws();
    if (p_ < e_ && *p_ == c) {
      ++p_;
      return true;
    }
    return false;
  }
  bool end() {
    ws();
    return p_ == e_;
  }
  bool word(const char* w) {
    const size_t n = std::strlen(w);
    if ((size_t)(e_ - p_) >= n && std::memcmp(p_, w, n) == 0) {
      p_ += n;
      return true;
    }
    return false;
  }
  bool str(std::string* out) {
    if (!lit('"')) return false;
    while (p_ < e_ && *p_ != '"') {
      char c = *p_++;
      if ((unsigned char)c < 0x20) return false;
      if (c == '\\') {
        if (p_ >= e_) return false;
        const char d = *p_++;
        switch (d) {
          case '"': case '\\': case '/': c = d; break;
          case 'b': c = '\b'; break;
          case 'f': c = '\f'; break;
          case 'n': c = '\n'; break;
          case 'r': c = '\r'; break;
          case 't': c = '\t'; break;
          case 'u':
            if (e_ - p_ < 4) return false;
            for (int i = 0; i < 4; ++i)
              if (!std::isxdigit((unsigned char)p_[i])) return false;
            p_ += 4;
            c = '?';  // keys of the cache are ASCII; anything else never matches
            break;
          default: return false;
        }
      }
      if (out) out->push_back(c);
    }
    if (p_ >= e_) return false;
    ++p_;
    return true;
  }
  bool num(double* v) {
    ws();
    const char* s = p_;
    while (p_ < e_ && (std::isdigit((unsigned char)*p_) || *p_ == '-' || *p_ == '+' ||
                       *p_ == '.' || *p_ == 'e' || *p_ == 'E'))
      ++p_;
    if (p_ == s || p_ - s > 64) return false;
    char buf[72];
    std::memcpy(buf, s, (size_t)(p_ - s));
    buf[p_ - s] = '\0';
    char* endp = nullptr;
    const double x = std::strtod(buf, &endp);
    if (endp != buf + (p_ - s) || !std::isfinite(x)) return false;
    if (v) *v = x;
    return true;
  }
  bool array(std::vector<double>* nums, bool* all_num) {
    if (!lit('[')) return false;
    if (lit(']')) return true;
    for (;;) {
      const char c = peek();
      if (c == '-' || (c >= '0' && c <= '9')) {
        double x;
        if (!num(&x)) return false;
        if (nums) nums->push_back(x);
      } else {
        if (all_num) *all_num = false;
        if (!skip()) return false;
      }
      if (lit(',')) continue;
      return lit(']');
    }
  }
  bool object_skip() {
    if (!lit('{')) return false;
    if (lit('}')) return true;
    for (;;) {
      if (!str(nullptr) || !lit(':') || !skip()) return false;
      if (lit(',')) continue;
      return lit('}');
    }
  }
  bool skip() {
    if (++depth_ > 64) return false;
    bool ok;
    const char c = peek();
    if (c == '{') ok = object_skip();
    else if (c == '[') ok = array(nullptr, nullptr);
    else if (c == '"') ok = str(nullptr);
    else if (c == 't') ok = word("true");
    else if (c == 'f') ok = word("false");
    else if (c == 'n') ok = word("null");
    else ok = num(nullptr);
    --depth_;
    return ok;
  }
  // {"tile": [mt, nbt, nbp, kres, sgw], ...}
  bool entry(TuneEntry* e, bool* good) {
    if (!lit('{')) return false;
    *good = false;
    if (lit('}')) return true;
    for (;;) {
      std::string k;
      if (!str(&k) || !lit(':')) return false;
      if (k == "tile" && peek() == '[') {
        std::vector<double> v;
        bool all_num = true;
        if (!array(&v, &all_num)) return false;
        bool ints = all_num && v.size() == 5;
        for (size_t i = 0; ints && i < v.size(); ++i)
          ints = v[i] == std::floor(v[i]) && v[i] >= -1024 && v[i] <= 1048576;
        if (ints) {
          e->tile = Tile{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
          e->sgw = (int32_t)v[4];
          *good = true;
        }
      } else if (!skip()) {
        return false;
      }
      if (lit(',')) continue;
      return lit('}');
    }
  }
};

}  // namespace

int parse_tune_cache(const char* text, size_t len, std::vector<TuneEntry>* out) {
  if (!text || !out) return -1;
  std::vector<TuneEntry> got;
  Reader r(text, len);
  if (!r.top(&got)) return -1;
  out->insert(out->end(), got.begin(), got.end());
  return (int)got.size();
}

}  // namespace bf
