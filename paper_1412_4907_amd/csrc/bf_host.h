// bf_host.h -- host-side logic of the beamformer library that needs no HIP:
// argument checks, the work schedule of a plan, the default tile choice, and
// the reader of the autotuner's tile cache.  bf_api.cpp builds on it, and a
// CPU-only test build compiles it with address and undefined-behaviour
// sanitizers.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/bf.h"
#include "bf_tiles.h"

namespace bf {

// Limits of bf_plan_create_ex.
constexpr int32_t kMaxN = 4096;
constexpr int32_t kMaxB = 65536;
constexpr int32_t kMaxC = 1 << 24;
constexpr int64_t kMaxT = (int64_t)1 << 40;
constexpr size_t kLdsMax = 160 * 1024 - 256;  // dynamic LDS; the rest is static

// The facts about a plan that the host logic needs.
struct Shape {
  int32_t N = 0, C = 0, B = 0, I = 0;
  int64_t T = 0;
  int prec = 0;          // bf_precision_t
  uint32_t flags = 0;    // BF_ACCUMULATE | BF_INPUT_4BIT | BF_OUTPUT_COMPLEX
  bool in4 = false;      // 4-bit input (one byte per antenna sample)
  bool cx = false;       // complex FP16 beam output
  bool vec16 = true;     // 2N % 16 == 0: a lane's 16 K values are one 16-byte load
  int32_t Bpad = 0;      // B rounded up to 16
  int32_t Kpad = 0;      // 2N rounded up to kChunk
  int mode = 0;          // Mode
  int n_cu = 256;        // compute units of the device
};

// Validates a plan request and fills *out.  Returns BF_OK,
// BF_ERR_INVALID_ARG (sizes, precision, unknown flags, complex output with
// I != 1 or with BF_ACCUMULATE) or BF_ERR_UNSUPPORTED (4-bit input with
// N % 8 != 0).
int make_shape(int32_t N, int32_t C, int32_t B, int64_t T, int32_t I, int prec, uint32_t flags,
               int n_cu, Shape* out);

int es_of(int prec);
int mode_of(int32_t I);
// Dynamic LDS of a beam range of nbt 16-beam tiles (weight rows for all K),
// in the storage precision and split into the MFMA operand parts (FP32: three
// BF16 parts, 6 bytes per weight), padded per 64-wide chunk.
size_t lds_bytes(int prec, int32_t Kpad, int nbt);
size_t split_lds_bytes(int prec, int32_t Kpad, int nbt);
// Dynamic LDS of a form: split rows for the register-resident and streamed
// forms, none when the weights are read from device memory.
size_t tile_lds(int prec, int32_t Kpad, Tile t);
// Row-tile schedule for integration I: MFMA row tiles per store group (G),
// per window (QI) and store groups per channel (SG).
void schedule(int32_t I, int64_t T, int32_t* G, int32_t* QI, int32_t* SG);
bool same_tile(const Tile& a, const Tile& b);
// Whether the shape's byte offsets fit the 32-bit buffer offsets of the
// register-resident and streamed forms at a width of nbt beam tiles: they count
// from a wave's first voltage row (over as few store groups as it may have) and
// from a beam range's first output row, so a channel may be longer.
bool buffer_shape(const Shape& s, int nbt);
// The store groups per wave of a run under form f where sgw are asked for: as
// many of them as its offsets reach.
int32_t wave_sgw(const Shape& s, const Tile& f, int32_t sgw);
// Whether the register-resident form (2N <= 64) can run the shape.
bool fast_ok(const Shape& s);
// The streamed form's tile for the shape (BF_TILE_LIST_STREAM), with weights
// of at most lds_cap bytes; false if there is none.
bool stream_tile(const Shape& s, size_t lds_cap, Tile* t);
// The compiled form that runs tile name t of the shape: t itself, or what
// replaced it.
Tile form_of(const Shape& s, Tile t);
// Whether the single-set kernel compiled for this shape's input, output
// and row width carries tile t.
bool tile_exists(const Shape& s, Tile t);
// Whether a compiled tile can run the shape (K and LDS budget).
bool tile_ok(const Shape& s, Tile t);
// Work units (workgroups) of one run under (t, sgw).
int64_t units_for(const Shape& s, Tile t, int32_t sgw);
// Store groups per wave of one run under form t.
int32_t choose_sgw(const Shape& s, Tile t);
// The default tile and store groups per wave.
void choose_tile(const Shape& s, Tile* t, int32_t* sgw);
// BF_OK if (t, sgw) can run the shape; BF_ERR_UNSUPPORTED (tile not
// compiled, K or LDS) or BF_ERR_INVALID_ARG (sgw).
int check_tile(const Shape& s, Tile t, int32_t sgw);
// Every single-set tile compiled for the shape's form, in list order.
std::vector<Tile> compiled_tiles(const Shape& s);
// One name for each form that runs the shape: the form's own where it has one.
// (An FP16 plan of 32 antennas at I = 1 has 20 names for 12 forms; timing all of
// them would time one kernel eight times and keep its luckiest run.)
std::vector<Tile> offered_tiles(const Shape& s);
// The variants the persistent batching kernel carries.
std::vector<Tile> multi_tiles();
// Variants of the eight-wave batching kernels (BF_TILE_LIST_WIDE order).
std::vector<Tile> wide_tiles();
// Whether the shape's sets of a table with eight-wave launches are accepted
// (also: whether the tile names with kres == -2 are offered).
bool wide_shape(const Shape& s);
// The four-wave batching variant (index into BF_TILE_LIST_MULTI) for a set,
// with at most lds_cap bytes of LDS: the tile `own` if the kernel carries its
// form (null: none asked for), else the widest beam range the set's beams fill
// that leaves two workgroups per CU; -1: none.
int multi_variant(const Shape& s, const Tile* own, size_t lds_cap);
// The eight-wave batching variant (index into BF_TILE_LIST_WIDE) for a set: the
// widest beam range whose weights fit lds_cap and that the set's beams fill
// beyond one of half the width; -1: none.  *sgw: its store groups per wave: as
// much of the channel's time range as spreads over the eight waves (at least one
// MT-aligned step each), so that no wave of a unit idles on a short block and a
// long block is split into as few units as that allows, each staging its
// weights once (a 12-set batch against each set's own count capped the same
// way: 19.05-19.10 -> 18.76-18.80 ms).
int wide_variant(const Shape& s, size_t lds_cap, int32_t* sgw);
// A set of a batch and its plan's tile.
struct BatchSet {
  const Shape* s;
  Tile tile;
  int32_t sgw;
};
// Which sets of a batch (16-byte rows) run in a persistent launch of the
// eight-wave streamed form, the others in the four-wave launch behind it.  True
// if any does.
// One launch of the eight-wave form takes them all where every set has more than
// two chunks of K and either the sets whose own tile it is have two units per CU
// (FP32, N 256 / 256 / 304, 64, 16 and 8 channels, I = 16: 834 -> 403 us), or, in
// 16 bits at I % 4 == 0, the sets for whose four beam tiles two four-wave
// workgroups do not fit a CU make up 3/4 unit per CU there (N 200 and 256, 32
// channels, FP16: I = 16 143 -> 109 us, I = 64 151 -> 135, but 178 -> 186 at I = 1
// and 138 -> 145 at I = 2; with 64 units of N = 256 the four-wave launch stays: 41
// against 59).
// Else two launches, where both fill the device several times: each drains on
// its own (four sets of 10 to 112 channels: 308 us split, 110 together).
bool wide_sets(const BatchSet* sets, int n, bool* wide);
// Modelled cycles of one unit of form f with v store groups per wave.
double unit_cycles(const Shape& s, Tile f, int32_t v, int wg);

// Bytes of one block of voltages, and of one run's output.
uint64_t input_bytes(const Shape& s);
uint64_t output_bytes(const Shape& s);
// Whether byte ranges [a, a + na) and [b, b + nb) share a byte.
bool ranges_overlap(const void* a, uint64_t na, const void* b, uint64_t nb);

// ---- tile cache written by the autotuner ----
// Key of a shape: precision, input and output form, N, I exactly; B, C and
// T as the largest power of two not above them (their effect on the best
// tile is through the number of work units, which changes slowly); batch
// selects the batching kernel's own entry.
std::string tune_key(const Shape& s, bool batch, const char* arch = "gfx950");
struct TuneEntry {
  std::string key;
  Tile tile;
  int32_t sgw;
};
// Reads the JSON object the autotuner writes ({"key": {"tile": [mt, nbt,
// nbp, kres, sgw], ...}, ...}); entries without a well-formed five-integer
// "tile" are skipped.  Returns the number of entries appended to *out, or -1
// if the text is not a JSON object (out is then unchanged).
int parse_tune_cache(const char* text, size_t len, std::vector<TuneEntry>* out);

}  // namespace bf
