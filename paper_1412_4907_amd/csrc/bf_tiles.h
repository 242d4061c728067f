// bf_tiles.h -- constants, integration classes and the compiled tile
// variants of the beamform kernel.  Plain C++ with no HIP dependency: the
// kernels (through bf_internal.h) and the host logic (bf_host.h) share it.
#pragma once

#include <stdint.h>

namespace bf {

constexpr int kMaxProbs = 16;   // beam sets per launch (kernel-argument table)
constexpr int kWaves = 4;       // waves per workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kWideWaves = 8;   // waves per workgroup of the eight-wave form
constexpr int kWideThreads = 64 * kWideWaves;
constexpr int kKresWide = -2;     // Tile::kres of the streamed form, eight waves: the name it
                                  // has for FP16/BF16 with I == 1 or I % 4 == 0
constexpr int kKresStream8 = -3;  // streamed form, eight waves
constexpr int kKresStream4 = -4;  // streamed form, four waves
constexpr int kXcds = 8;        // accelerator dies (XCDs), each with its own L2
constexpr int kQueueStride = 16;  // int32 slots between the per-XCD queue counters
// one persistent launch's counters: a queue per XCD, and the workgroups done
constexpr int kQueueInts = (kXcds + 1) * kQueueStride;
constexpr int kChunk = 64;      // real K elements (32 antennas) per chunk
constexpr int kLdsPad = 16;     // bytes added to each LDS weight row

// Integration classes; each is a separate kernel instantiation:
// I == 1, I == 2, I >= 3 with I % 4 != 0 (padded windows), I % 4 == 0;
// and complex beam output (no detection, I == 1 row mapping).
enum Mode : int { kModeI1 = 0, kModeI2 = 1, kModeGen = 2, kModeGen4 = 3, kModeCx = 4 };

// Tile variant of the beamform kernel.
struct Tile {
  int mt;    // 16-row MFMA tiles per wave step
  int nbt;   // 16-beam tiles per workgroup beam range
  int nbp;   // 16-beam tiles per accumulator pass
  int kres;  // K chunks held in registers per wave step (1), or the form (below)
};

// Waves that share one work unit's staged weights.
constexpr int waves_of(Tile t) {
  return t.kres == kKresWide || t.kres == kKresStream8 ? kWideWaves : kWaves;
}

// Tile names (MT, NBT, NBP, KRES).  KRES 1 and 2 serve plans with
// Kpad / 64 <= KRES; KRES == 0 streams K with the unit's weights in LDS in
// the storage precision; KRES == -1 streams K with the weights read from
// device memory (any K: arrays whose weight rows do not fit LDS); -2, -3 and
// -4 are the streamed form.  A name says what a plan may be given
// (bf_plan_set_tile, tile caches); form_of (bf_host.h) maps it to one of the
// compiled forms, several names to one where a form replaced others.  The
// generic list serves plans whose 2N is not a multiple of 16.
#define BF_TILE_LIST_VEC16                                                        \
  BF_TILE(8, 8, 1, 1) BF_TILE(4, 8, 2, 1) BF_TILE(4, 8, 1, 1) BF_TILE(8, 4, 1, 1)  \
  BF_TILE(4, 4, 1, 1) BF_TILE(4, 8, 1, 2) BF_TILE(4, 4, 1, 2) BF_TILE(4, 8, 2, 0)  \
  BF_TILE(4, 4, 2, 0) BF_TILE(4, 2, 2, 0) BF_TILE(4, 2, 1, 0) BF_TILE(4, 1, 1, 0)  \
  BF_TILE(4, 4, 4, 0) BF_TILE(4, 2, 2, -1) BF_TILE(8, 1, 1, -1)
#define BF_TILE_LIST_GENERIC                                                      \
  BF_TILE(4, 8, 2, 0) BF_TILE(4, 4, 4, 0) BF_TILE(4, 1, 1, 0) BF_TILE(4, 2, 2, -1)
// Names for 4-bit input.
#define BF_TILE_LIST_IN4                                                          \
  BF_TILE(4, 8, 1, 1) BF_TILE(4, 8, 2, 1) BF_TILE(4, 4, 1, 1) BF_TILE(4, 8, 1, 2)  \
  BF_TILE(4, 8, 2, 0) BF_TILE(4, 4, 2, 0) BF_TILE(4, 2, 2, 0) BF_TILE(4, 1, 1, 0)  \
  BF_TILE(4, 4, 4, 0) BF_TILE(4, 2, 2, -1)
// Names for complex beam output (16-byte rows; byte-load plans use the
// generic list).
#define BF_TILE_LIST_CX                                                           \
  BF_TILE(4, 8, 1, 1) BF_TILE(4, 4, 1, 1) BF_TILE(4, 8, 1, 2) BF_TILE(4, 8, 2, 0)  \
  BF_TILE(4, 2, 2, 0) BF_TILE(4, 1, 1, 0) BF_TILE(4, 4, 4, 0) BF_TILE(4, 2, 2, -1)
// Compiled forms.  General (any size; BYTES is its byte-load list), with more
// than two beam tiles per range in 16 bits four in one pass, in FP32 (whose
// fragments and sums would not fit the registers) two per pass:
#define BF_TILE_LIST_GENERAL                                                      \
  BF_TILE(4, 8, 2, 0) BF_TILE(4, 4, 2, 0) BF_TILE(4, 4, 4, 0) BF_TILE(4, 2, 2, 0)  \
  BF_TILE(4, 1, 1, 0) BF_TILE(4, 2, 2, -1) BF_TILE(8, 1, 1, -1)
#define BF_TILE_LIST_BYTES                                                        \
  BF_TILE(4, 8, 2, 0) BF_TILE(4, 4, 4, 0) BF_TILE(4, 1, 1, 0) BF_TILE(4, 2, 2, -1)
// Register-resident pipelined form (2N <= 64):
#define BF_TILE_LIST_FAST                                                         \
  BF_TILE(4, 8, 1, 1) BF_TILE(4, 6, 1, 1) BF_TILE(4, 4, 1, 1) BF_TILE(4, 2, 1, 1)  \
  BF_TILE(4, 1, 1, 1)
// Streamed form (every beam tile of the range in one pass: NBP == NBT):
#define BF_TILE_LIST_STREAM                                                       \
  BF_TILE(4, 4, 4, -3) BF_TILE(4, 2, 2, -3) BF_TILE(4, 1, 1, -3)                   \
  BF_TILE(4, 4, 4, -4) BF_TILE(4, 2, 2, -4) BF_TILE(4, 1, 1, -4)
// The persistent batching kernels' variants: eight waves, and four waves
// (16-byte rows).
#define BF_TILE_LIST_WIDE BF_TILE(4, 4, 4, -3) BF_TILE(4, 2, 2, -3) BF_TILE(4, 1, 1, -3)
#define BF_TILE_LIST_MULTI                                                        \
  BF_TILE(4, 8, 1, 1) BF_TILE(4, 4, 1, 1) BF_TILE(4, 4, 4, -4) BF_TILE(4, 2, 2, -4) \
  BF_TILE(4, 1, 1, -4) BF_TILE(4, 1, 1, 0)

}  // namespace bf
