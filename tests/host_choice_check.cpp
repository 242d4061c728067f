// Choices of the host logic whose lines were drawn by measurement, built for the
// CPU (tests/test_host_choice.py).  Prints "OK ..." and exits 0, or names the
// first failed check and exits 1.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "bf_host.h"

using bf::Shape;
using bf::Tile;

static int g_checks = 0;

#define CHECK(cond)                                                               \
  do {                                                                            \
    ++g_checks;                                                                   \
    if (!(cond)) {                                                                \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond);                \
      return 1;                                                                   \
    }                                                                             \
  } while (0)

static Tile chosen(int N, int C, int B, int64_t T, int I, int prec, uint32_t flags = 0,
                   int32_t* sgw_out = nullptr) {
  Shape s;
  Tile t{0, 0, 0, 0};
  int32_t sgw = 0;
  if (bf::make_shape(N, C, B, T, I, prec, flags, 256, &s) != BF_OK) return t;
  bf::choose_tile(s, &t, &sgw);
  if (bf::check_tile(s, t, sgw) != BF_OK) return Tile{0, 0, 0, 0};
  if (sgw_out) *sgw_out = sgw;
  return t;
}

// Where two beam tiles' weights fit LDS only without padding per chunk, and
// byte-load rows whose weights leave one workgroup per CU.
static int check_large_arrays() {
  for (int prec : {BF_FP16, BF_BF16})
    for (int N : {552, 576, 600, 608})
      for (int I : {1, 2, 16, 64}) {
        const Tile t = chosen(N, 27, 256, 7680, I, prec);
        CHECK(t.mt == 4 && t.nbt == 2 && t.nbp == 2 && t.kres == 0);
        CHECK(chosen(N, 27, 16, 7680, I, prec).kres < -1);  // one beam tile: streamed
      }
  for (int N : {544, 552, 608, 616})
    CHECK(chosen(N, 27, 256, 7680, 5, BF_FP16).kres < -1);  // dummy rows: streamed
  CHECK(chosen(560, 8, 395, 1344, 64, BF_FP16).kres < -1);  // 104 units for 256 CUs
  CHECK(chosen(544, 27, 256, 7680, 64, BF_FP16).kres < -1);  // two streamed tiles fit
  CHECK(chosen(544, 27, 256, 7680, 64, BF_FP16).nbt == 2);
  CHECK(chosen(616, 27, 256, 7680, 64, BF_FP16).kres < -1);
  for (int I : {1, 5, 64}) {
    CHECK(chosen(1121, 14, 256, 7680, I, BF_FP16).kres == -1);
    CHECK(chosen(1121, 14, 16, 7680, I, BF_BF16).kres == (I == 64 ? 0 : -1));  // 112 units
    CHECK(chosen(601, 14, 256, 7680, I, BF_FP32).kres == -1);
    CHECK(chosen(1120, 14, 256, 7680, I, BF_FP16).kres == 0);  // 16-byte rows keep LDS
  }
  // no more units than CUs: LDS
  CHECK(chosen(1121, 2, 16, 49984, 64, BF_FP16).kres == 0);
  CHECK(chosen(1121, 2, 16, 50000, 16, BF_BF16).kres == 0);
  CHECK(chosen(1121, 2, 35, 50000, 16, BF_BF16).kres == -1);
  CHECK(chosen(601, 2, 35, 49984, 64, BF_FP32).kres == 0);
  CHECK(chosen(601, 2, 160, 49984, 64, BF_FP32).kres == -1);
  return 0;
}

struct Set {
  int N, C, B, W;
  bool stream8;  // asks for tile (4, 1, 1, -3, 4)
};

// 0: no set in the eight-wave launch, 1: some, 2: all
static int wide_of(const Set* sets, int n, int I, int prec) {
  Shape s[16];
  bf::BatchSet b[16];
  bool wide[16];
  for (int i = 0; i < n; ++i) {
    if (bf::make_shape(sets[i].N, sets[i].C, sets[i].B, (int64_t)sets[i].W * I, I, prec, 0, 256,
                       &s[i]) != BF_OK)
      return -1;
    b[i].s = &s[i];
    if (sets[i].stream8) {
      b[i].tile = Tile{4, 1, 1, -3};
      b[i].sgw = 4;
      if (bf::check_tile(s[i], b[i].tile, 4) != BF_OK) return -1;
    } else {
      bf::choose_tile(s[i], &b[i].tile, &b[i].sgw);
    }
  }
  if (!bf::wide_sets(b, n, wide)) return 0;
  int k = 0;
  for (int i = 0; i < n; ++i) k += wide[i];
  return k == n ? 2 : 1;
}

// The batches of tests/test_gpu_batch_wide.py take the eight-wave launch; and the
// shapes the rule was drawn from.
static int check_wide_batches() {
  const Set all[] = {{136, 520, 16, 32, true}, {200, 520, 10, 20, true}};
  const Set mixed[] = {{136, 520, 16, 32, true}, {200, 520, 10, 20, true},
                       {16, 1030, 16, 32, false}, {32, 1030, 30, 6, false}};
  const Set shared[] = {{136, 520, 16, 32, true}, {136, 520, 40, 32, true},
                        {136, 520, 5, 32, true}};
  for (int prec : {BF_FP16, BF_BF16, BF_FP32})
    for (int I : {1, 2, 10, 16}) {
      CHECK(wide_of(all, 2, I, prec) == 2);
      CHECK(wide_of(mixed, 4, I, prec) == 1);
      CHECK(wide_of(shared, 3, I, prec) == 2);
    }
  const Set pair[] = {{200, 32, 300, 240, false}, {256, 32, 100, 240, false}};
  CHECK(wide_of(pair, 2, 16, BF_FP16) == 2);
  const Set pair1[] = {{200, 32, 300, 3840, false}, {256, 32, 100, 3840, false}};
  CHECK(wide_of(pair1, 2, 1, BF_FP16) == 0);
  const Set one[] = {{256, 64, 64, 120, false}};
  CHECK(wide_of(one, 1, 16, BF_FP16) == 0);
  const Set tiny[] = {{256, 8, 64, 1920, false}};
  CHECK(wide_of(tiny, 1, 1, BF_FP16) == 0);
  const Set f32[] = {{256, 64, 300, 240, false}, {256, 16, 16, 60, false}, {304, 8, 40, 60, false}};
  CHECK(wide_of(f32, 3, 16, BF_FP32) == 2);
  const Set small_mix[] = {{120, 8, 151, 1762, false}, {160, 9, 394, 93, false},
                           {24, 101, 344, 263, false}, {200, 77, 18, 239, false}};
  CHECK(wide_of(small_mix, 4, 8, BF_BF16) == 0);
  return 0;
}

// Channels past 2 GiB: offsets count from a wave's first row and a beam range's
// first output row.
static int check_long_channels() {
  const int64_t T = 35651520;  // 32 antennas: 2.28 GB
  int32_t sgw = 0;
  Tile t = chosen(32, 1, 64, T, 16, BF_FP16, 0, &sgw);
  CHECK(t.kres == 1 && t.nbt > 1);
  t = chosen(32, 1, 64, T, 10, BF_BF16);
  CHECK(t.kres == bf::kKresStream4 && t.nbt == 4);
  CHECK(chosen(33, 1, 64, T, 16, BF_FP16).kres < -1);
  CHECK(chosen(32, 1, 64, 2 * T, 16, BF_FP16, BF_INPUT_4BIT).kres == 1);
  // 64 output rows past the offsets: 64-bit rows in 16 bits, narrower ranges else
  for (int I : {1, 2}) CHECK(chosen(32, 1, 64, T, I, BF_FP16).kres == 0);
  CHECK(chosen(32, 1, 64, T, 2, BF_FP32).kres == bf::kKresStream4);
  t = chosen(32, 1, 64, T, 4, BF_FP16);
  CHECK(t.kres == 1 && t.nbt == 2);
  t = chosen(8, 1, 64, 142606080, 16, BF_FP16);
  CHECK(t.kres == 1 && t.nbt == 2);
  // store groups per wave: as asked for while the channel fits, else as many as
  // the offsets reach, in whole wave steps
  int cut = 0;
  for (int N : {1, 8, 32, 33, 256, 4096})
    for (int I : {1, 2, 3, 16, 1000})
      for (int64_t T1 : {(int64_t)6000, (int64_t)6000000, (int64_t)1500000000})
        for (int B : {1, 64}) {
          Shape s;
          if (bf::make_shape(N, 1, B, T1, I, BF_FP16, 0, 256, &s) != BF_OK) continue;
          for (int nbt : {1, 4}) {
            if (!bf::buffer_shape(s, nbt)) continue;
            const Tile f{4, nbt, nbt, bf::kKresStream4};
            const int32_t base = I == 1 ? 4 : I == 2 ? 2 : 1;
            for (int32_t g : {base, 12, 1 << 20}) {
              const int32_t v = bf::wave_sgw(s, f, g);
              CHECK(v >= base && v <= g && (v == g || v % base == 0));
              const int64_t rows = std::min(T1, (int64_t)v * 16 * I);
              CHECK((rows + 16 * (int64_t)I) * 2 * N < ((int64_t)1 << 31));
              CHECK(std::min(B, 16 * nbt) * (T1 / I) * 4 < ((int64_t)1 << 31));
              cut += v < g;
            }
          }
        }
  CHECK(cut > 20);
  return 0;
}

// Tile candidates: one name per form, and every form that a name stands for.
static int check_offered() {
  int fewer = 0;
  for (int prec = 0; prec < 3; ++prec)
    for (int N : {1, 16, 32, 33, 40, 64, 256, 600, 1248, 4096})
      for (int B : {4, 33, 128, 512})
        for (int I : {1, 2, 5, 16})
          for (uint32_t fl : {0u, (uint32_t)BF_ACCUMULATE, (uint32_t)BF_INPUT_4BIT,
                              (uint32_t)BF_OUTPUT_COMPLEX}) {
            Shape s;
            if (bf::make_shape(N, 3, B, 4800, I, prec, fl, 256, &s) != BF_OK) continue;
            const std::vector<Tile> v = bf::offered_tiles(s);
            CHECK(!v.empty());
            for (size_t i = 0; i < v.size(); ++i) {
              CHECK(bf::tile_ok(s, v[i]));
              for (size_t j = 0; j < i; ++j)
                CHECK(!bf::same_tile(bf::form_of(s, v[i]), bf::form_of(s, v[j])));
            }
            size_t names = 0;
            for (const Tile& t : bf::compiled_tiles(s)) {
              if (!bf::tile_ok(s, t)) continue;
              ++names;
              bool there = false;
              for (const Tile& o : v)
                there = there || bf::same_tile(bf::form_of(s, t), bf::form_of(s, o));
              CHECK(there);
            }
            fewer += v.size() < names;
          }
  CHECK(fewer > 100);
  return 0;
}

int main() {
  if (check_offered()) return 1;
  if (check_large_arrays() || check_wide_batches() || check_long_channels()) return 1;
  std::printf("OK %d checks\n", g_checks);
  return 0;
}
