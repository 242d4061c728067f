// Choices of the host logic whose lines were drawn by measurement, built for the
// CPU (tests/test_host_choice.py).  Prints "OK ..." and exits 0, or names the
// first failed check and exits 1.
#include <cstdio>

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
  CHECK(chosen(544, 27, 256, 7680, 64, BF_FP16).kres < -1);  // two streamed tiles fit
  CHECK(chosen(544, 27, 256, 7680, 64, BF_FP16).nbt == 2);
  CHECK(chosen(616, 27, 256, 7680, 64, BF_FP16).kres < -1);
  for (int I : {1, 5, 64}) {
    CHECK(chosen(1121, 14, 256, 7680, I, BF_FP16).kres == -1);
    CHECK(chosen(1121, 14, 16, 7680, I, BF_BF16).kres == -1);
    CHECK(chosen(601, 14, 256, 7680, I, BF_FP32).kres == -1);
    CHECK(chosen(1120, 14, 256, 7680, I, BF_FP16).kres == 0);  // 16-byte rows keep LDS
  }
  return 0;
}

int main() {
  if (check_large_arrays()) return 1;
  std::printf("OK %d checks\n", g_checks);
  return 0;
}
