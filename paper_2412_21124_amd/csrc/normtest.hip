// libnormtest: norm-test statistics pass fused with AdamW, hand-written for gfx950 (MI355X).
//
// One streaming kernel (k_step) reads the J gradient rows and w, m, v once, writes w, m, v once and
// leaves five fp64 values per fixed-size tile of coordinates (the sums A, B, C, the count of coordinates
// failing the coordinate-wise form of the test, and their largest ratio); k_finalize or k_reduce_end then add
// the tile partials in double-double arithmetic and take Alg. 1's decision on the device (steps of few tiles, and AdamW only,
// need no second kernel: k_step_end).  The partials stay in the caller's workspace
// behind a small record of the step, from which k_layer_stats can regroup them into a per-layer table.
// k_adamw_gbar is the second phase of the gradient-clipped variant.  The
// path is bound by HBM bandwidth (about two lane-operations per byte), so there is no MFMA here: the work is
// fully coalesced 8- and 16-byte accesses, fp32 per-coordinate arithmetic, fp64 accumulation and sums across a
// wave by register swaps and row moves.  Launch shapes (block size, sweeps per tile, coordinates per launch) differ per class of
// call and were chosen by measurement; see tile_cfg() and the NT_CHUNK_* constants.  Two things about the memory
// system shape the host side: blocks that start together stay in step for a while and are served faster than an
// even mix of loads and stores, so a long vector is walked by several launches; and writes sprinkled among many
// reads cost several times their volume, so with more than 16 rows (tile_multi), and in long vectors from 28
// bytes of gradient per coordinate on (tile_defer), a block updates the state of its whole tile only after it
// has read all the rows.
//
// Numerics.  The centred sum C = sum_j (g_j - gbar)^2 is formed directly from the J values of a
// coordinate held in registers, never as A - B/J (which cancels badly when the workers agree).  A
// rounding error e in gbar only adds J e^2 to a coordinate's centred sum because the cross term
// sums to zero.  More than 16 fp32 rows are taken 16 at a time, each chunk shifted by the
// running mean so far, and the chunks' means and centred sums are merged with the pairwise update
// M2 += M2_b + delta^2 n_a n_b / (n_a + n_b).  More than 16 bf16 rows, whose squares have 16 bits, are summed with their squares in
// fp64, where both are exact or nearly so, and C is the difference (centred).  Row sums are carried in fp64, so the mean handed to
// AdamW is correctly rounded even when the rows cancel.
// Per-lane sums leave fp32 after one group of 4 coordinates; everything above is fp64 in a fixed
// order, so results do not depend on the grid size and are reproducible bit for bit.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "normtest.h"

// Launch shapes, chosen by measurement on MI355X (block size, block sweeps per partial-sum tile).
#define NT_BLOCK 1024            // J <= 16, fused step: one sweep of a large block per tile
#define NT_ITERS 1
#define NT_BLOCK_STATS 512       // J <= 16, statistics only: read-only and few bytes per lane, so smaller blocks
#define NT_ITERS_STATS 8         // that each walk a longer tile
#define NT_STATS_SHORT_COORDS (1ll << 21)  // ... in vectors shorter than this, the next shape (64 blocks of 512 threads
                                           // for 2^20 coordinates leave most of the chip idle: 18 -> 14 us at 8 rows)
#define NT_BLOCK_STATS_GBAR 512  // statistics that also store gbar (phase 1 of the clipped variant): one write
#define NT_ITERS_STATS_GBAR 2    // stream moves the optimum to shorter tiles
#define NT_BLOCK_ADAMW 1024      // J <= 16, AdamW only (test skipped)
#define NT_ITERS_ADAMW 1
#define NT_BLOCK_LARGE 128       // J > 16 (rows are walked inside each sweep), every mode that writes per coordinate:
#define NT_ITERS_LARGE 16        // a block walks the rows of all its sweeps first and writes for all of them afterwards,
#define NT_GENS_LARGE 1          // and a launch holds this many generations of blocks (CUs x blocks per CU)
#define NT_LDS_PAD_LARGE 1024    // LDS bytes on top of the 32 KB of means: four blocks per CU in every mode (five are slower)
#define NT_FEW_ROWS 20           // 17 .. this many rows: the same tile as 256 threads x 8 sweeps (fused step +9 % at 17 rows,
#define NT_BLOCK_FEW 256         // +7 % at 20, +3 % at 24 but AdamW only -1 % there, -1.5 % at 28): the walk is short
#define NT_ITERS_FEW 8           // there, and a block's life with it
// Up to 16 rows with at least NT_DEFER_ROW_BYTES of gradient per coordinate (14 bf16 or 7 fp32 rows; AdamW only:
// NT_DEFER_ROW_BYTES_ADAMW, 10 or 5 rows), in a vector of at least NT_DEFER_COORDS coordinates: a step that writes
// per coordinate runs like the many-row one, rows in registers but the update deferred and one generation of blocks
// per launch (+2 .. +8 % there; with fewer bytes per coordinate, or fewer than some eight generations, the
// interleaved class is as fast or faster).
#define NT_DEFER_ROW_BYTES 28
#define NT_DEFER_ROW_BYTES_ADAMW 20
#define NT_DEFER_COORDS (1ll << 26)
#define NT_BLOCK_DEFER 128
#define NT_ITERS_DEFER 16
#define NT_DEFER_UNROLL 1        // row sweeps in flight per lane in that class
#define NT_GENS_DEFER 1          // generations of blocks per launch in that class (two: -7 .. -10 %)
// J > 16, modes that write per coordinate: the shapes above where a generation of blocks (NT_GENERATION coordinates: four blocks on each
// of 256 CUs) is nearly full, or enough of the one after the first or second (generations_pay); else one launch of short tiles, of
// which the chip takes any number (512 rows, d = 2^18: 607 -> 92 us).
#define NT_GENERATION (1ll << 23)
#define NT_PAUSE_ROWS 48         // bf16 rows from which the walk pauses between chunks (chunk_pause)
#define NT_BLOCK_MANY_SHORT 256
#define NT_ITERS_MANY_SHORT 2
// J > 16, every mode, in short vectors, whose tiles leave each CU at most a block or two: the same tile as one sweep of
// 512 threads, so that a block walks the rows once.  Shape above -> this one, us: fused step of 17 / 64 / 512 bf16 rows at d =
// 100,003 9.2 / 18.7 / 103 -> 7.6 / 13.7 / 66, at 3e5 10.1 / 18.0 / 89.7 -> 8.4 / 14.0 / 62.7, at 5e5 11.8 / 19.4 / 95.4 -> 9.8 / 15.3 /
// 78.1, at 7e5 14.0 / 24.3 / 129 and 12.1 / 23.9 / 129, at 1e6 14.7 / 26.2 / 154 and 13.2 / 26.4 / 159, at 2e6 20 rows 23.7 and 25.5;
// of 17 / 32 / 128 fp32 rows at 30,000 10.1 / 11.9 / 30.8 -> 8.5 / 9.6 / 24.0, at 1e6 18.6 / 27.1 and 20.6 / 27.7; AdamW only, 64 bf16
// rows, 13.6 -> 10.0 at 3e5, 22.9 and 23.8 at 1e6.
#define NT_BLOCK_MANY_TINY 512
#define NT_ITERS_MANY_TINY 1
#define NT_MANY_TINY_COORDS (1ll << 19)
#define NT_MANY_TINY_COORDS_32 (1ll << 20)   // up to 32 bf16 rows, unless AdamW only
// J > 16, every mode, in the shortest vectors: tiles of 1024 coordinates.  A CU reads some 45 GB/s at most, whatever it has in flight, so
// what counts is how many of them have a tile.  bf16 rows: the waves of a block share the rows as well (tile_split), two of them up to
// 32 rows and four beyond, as one wave alone walks 512 rows in 32 steps of 2 us, most of it arithmetic.  fp32 rows: blocks of 256 threads.
// Shape above -> these, us: fused step of 17 / 64 / 128 / 512 bf16 rows at d = 20,001 7.8 / 13.7 / 21.4 / 66 -> 7.2 / 10.0 / 13.1 /
// 32, at 2^18 9.0 / 13.9 / 20.7 / 61 -> 8.3 / 11.4 / 16.5 / 46; of 17 / 64 / 512 fp32 rows at d = 100,003 9.0 / 15.8 / 84 -> 8.1 /
// 13.2 / 54; AdamW only, 64 bf16 rows 8.8 -> 6.1 at 100,003.  Beyond 2^18 coordinates some CUs have two tiles: 64 bf16 rows at 3e5 14.2
// and 15.1.
#define NT_SPLIT_TILE 1024
#define NT_SPLIT_COORDS (1ll << 18)
// Not so where one tile of NT_BLOCK_MANY_TINY threads holds the vector and there are few rows: a step with sums is then a kernel of one
// block, which counts nothing.  Tiles of 1024 -> one tile, us: fused step of 17 / 32 / 48 / 56 / 64 bf16 rows at d = 1025 6.8 / 7.2 / 8.8 / 9.0 /
// 9.4 -> 5.7 / 6.7 / 8.1 / 8.9 / 9.5, at 2048 6.7 / 7.3 / 8.6 / 8.6 / 9.0 -> 5.1 / 6.0 / 7.2 / 7.9 / 8.4; of 17 / 40 / 56 fp32 rows 6.8 / 8.4 / 9.7 -> 6.0 /
// 8.1 / 9.7 and 6.2 / 7.4 / 8.3 -> 5.0 / 6.8 / 8.1, statistics of 48 7.4 -> 7.9 and 7.4 -> 6.9.  Up to 1024 coordinates, one block either way: 17 / 24 /
// 32 bf16 rows 5.2 / 5.3 / 5.6 -> 4.9 / 5.1 / 5.7, statistics of 24 4.7 -> 4.4; fp32 rows are equal.
#define NT_ONE_TILE_ROWS 56
#define NT_ONE_TILE_ROWS_32 40   // fp32 rows
#define NT_ONE_TILE_ROWS_HALF 24 // bf16 rows, up to NT_SPLIT_TILE coordinates
#define NT_SPLIT 1000            // J_T of the kernels whose waves share the rows is NT_SPLIT + how many of them
#define NT_BLOCK_LARGE_STATS 256 // J > 16, statistics only otherwise (nothing written per coordinate): short tiles, so that a
#define NT_ITERS_LARGE_STATS 2   // vector of a few million coordinates still gives every CU several blocks
#define NT_MAX_GRID (1ll << 21)  // blocks per launch at most: HIP's limit is on the threads, 2^32 - 1
#define NT_COPY_BLOCKS_PER_CU 4096  // copy and yardstick: grid = min(blocks of work, CUs * this); blocks stride beyond that
// A long vector is walked by several launches of the step kernel, each over a run of consecutive tiles.  Blocks
// that start together move through their load and store phases together, so the memory system sees chip-wide
// bursts of reads and of writes instead of an even mix, which it serves faster; inside one long launch that
// lockstep drifts apart within some tens of block generations.  A kernel boundary restores it at the price of a
// drained machine for a few microseconds.  Coordinates per launch, by class (measured; 0: one launch):
#define NT_CHUNK_FULL (1ll << 26)        // J <= 16, fused step (2^25 .. 2^27 within 0.5 %, 2^24 -2 %, 2^28 -1 %)
#define NT_CHUNK_FULL_FEW (1ll << 25)    // ... of up to 8 bytes of rows, two blocks per CU (4 bf16 rows +1.2 .. 2 % against 2^27);
                                         // 5 to 7 bf16 rows, which take 2^26: 2^25 is -1.0 .. +0.8 %
#define NT_CHUNK_ADAMW (1ll << 25)       // J <= 16, AdamW only (+5 %)
#define NT_CHUNK_ADAMW_LONG (1ll << 24)  // ... in vectors of at least NT_LONG_COORDS, two blocks per CU
#define NT_LONG_COORDS (1ll << 28)
#define NT_CHUNK_STATS_GBAR (1ll << 27)  // J <= 16, statistics + stored gbar (+2 % on the clipped step)
#define NT_CHUNK_STATS 0                 // statistics only: nothing is written, nothing to gain
#define NT_CHUNK_ADAMW_GBAR (1ll << 25)  // AdamW from a stored gbar (second phase of the clipped step)
// J > 16, modes that write per coordinate: one generation of blocks per launch, see launch_step_shape

// Two blocks of 1024 threads fit a CU where a kernel has at most 64 vector registers: the fused step of up to 5 rows of either type
// and AdamW only of up to 16 bf16 or 10 fp32 rows.  In short vectors that hides latency; where a vector fills the chip several
// times over, one block at a time keeps the blocks in step and is served faster.  Asking for more than half of a CU's LDS sees to
// it (one_block_lds).  One against two, us: fused step of 4 fp32 rows 34.8 / 32.5 at d = 2^22, 121.4 / 120.4 at 2^24, 819 / 857
// at 124M, of 8 bf16 rows (where it keeps the next block from starting beside the last waves of a block) 35.5 / 34.7 at 2^22,
// 9740 / 9830 at 1.5e9; AdamW only, 8 bf16 rows 29.4 / 27.4 at 2^22, 61.2 / 59.1 at 2^23, 112 / 116 at 2^24, 194 / 200 at 3e7,
// 813 / 826 at 124M, 2013 / 1998 at 3e8; AdamW from a stored gbar +0.8 % from 6e7 on, -2 % at 1e7.  Up to 8 bytes of rows the
// fused step prefers two at any length (4 bf16 rows 28.6 / 25.9 at 2^22, 1683 / 1661 at 304.6M), AdamW only is indifferent.  5 bf16
// rows (10 bytes, two at any length): one is -4 % at 2^24, -0.6 % at 6e7 and 124M, +0.2 % at 3e8; 6 and 7 have the registers of one, and
// asking for the LDS too costs them 1 % up to 304.6M.
#define NT_ONE_BLOCK_LDS 82000
// Statistics that store the mean, up to 16 rows: the same with blocks of 512 threads, beyond 2^25 coordinates.  Three instead of the four
// per CU that the registers allow, two / three / four blocks, us: 5 bf16 rows 292 / 279 / 286 at d = 1.24e8, 149 / 140 / 141 at 6e7.  Two from 12
// bytes of rows on: 9 bf16 rows 310 / - / 323 at 9e7 (of three), 69 / - / 70 at 2^24; 4 fp32 rows 293 / - / 302 at 9e7; 6 bf16 rows 159 / 161 /
// 160 at 6e7, 341 / 347 / 354 at 1.3e8; 6 fp32 rows 425 / 434 / 436 at 9e7.  8 and 10 to 16 bf16 rows have the registers of two anyway, or
// are indifferent.
#define NT_TWO_BLOCK_LDS 56000
#define NT_THREE_BLOCK_LDS 42000
#define NT_HOLD_GBAR_COORDS (1ll << 25)

#define NT_VEC 4              // coordinates per lane and sweep: 16-byte fp32 accesses, 8-byte bf16 row loads
#define NT_TILE_MAX 16384     // every tile size divides this: the alignment that keeps shard results bit-identical
#define NT_AUX_BLOCK 1024     // threads per block of the AdamW-from-gbar, copy and yardstick kernels

#define NT_JCHUNK 16          // up to this many rows a coordinate's values are all held in registers
#define NT_SEGMENTS 4         // more than 16 bf16 rows are added up in up to this many segments (segment_rows)
#define NT_MCHUNK 16          // beyond that, rows are walked this many at a time (2 .. NT_JCHUNK + 1; 16 measured best)
#define NT_ROUND_TO_MAX (1ll << 31)  // bound on nt_hyper.round_to that keeps the rounding chain inside int64
#define NT_FIN_THREADS 256      // threads that add up tile or group partials
// Up to this many tiles a step's own last block adds up the tile partials (k_step_end), in one launch instead of two (3.7 us of
// host time).  Device time of the step, one launch against two: 4 fp32 rows 6.8 / 8.5 us at d = 5000, 7.2 / 8.5 at 2^18 and 8.9 /
// 10.5 at 2^20 (256 tiles); read-only statistics of 8 bf16 rows 5.7 / 8.0, 6.9 / 8.3 and 6.9 / 8.6; at 2^21 (512 tiles) the fused
// step of 4 and 8 bf16 rows 15.4 / 14.6 and 18.5 / 18.2, with a stored mean 8.5 / 8.6 and 10.6 / 10.8, where it is the second launch
// on the host that counts; at 2^22 14.1 / 13.4.  More than 16 rows: in the shortest vectors up to 256 tiles, 64 bf16 rows at 2^18 11.4 /
// 13.6; in the longer ones' tiles of 2048 coordinates, in kernels that live longer, up to 128: 17 / 64 rows at 2^19 (256 tiles) are
// equal, but 64 fp32 rows take 20.9 / 20.6 at 388,160 and 128 bf16 rows 56.2 / 55.7 at 1e6.
#define NT_TICKET_TILES 256
#define NT_TICKET_TILES_STATS 512
#define NT_TICKET_TILES_MANY 128
// Beyond this many tiles the blocks count themselves in NT_LEAVES counters, whose last ones then count themselves in one more: a
// counter takes some 10 ns per block, one after the other, and blocks that start together end together (256 tiles: fused step of 4
// fp32 rows 10.5 -> 8.9 us, statistics 8.2 -> 6.3; 128 tiles 7.9 -> 7.4 and 6.7 -> 6.3; 74 tiles 0.1 us slower; 16 or 32 leaves are no faster).
#define NT_LEAF_TILES 96
#define NT_LEAVES 8
#define NT_NSUM 4              // summed values per tile partial: A, B, C and the count of failing coordinates
#define NT_NV 5                // values per tile partial: the sums, then the largest coordinate-wise ratio
// Up to this many tiles one block adds up the tile partials (k_finalize); beyond, one block per group_tiles of them, of which the last
// to finish adds up the groups (k_reduce_end).  The launch alone takes 1.3 us and the chain of one block 1.5; a block reads some 45 GB/s,
// 40 bytes a tile, and the counting costs 1.9 us.  What a step takes beyond its streaming kernel, us, one block / groups: 512 tiles 3.3,
// 1024 3.8 / 5.7, 2048 4.8 / 5.0, 4096 7.0 / 5.4; 7325 tiles 5.1, in groups of 2048 and a second kernel for the groups 7.1.
#define NT_DIRECT_TILES 2560
// Tiles per group: enough groups to read the partials side by side, and not so many that they queue at the counter.
inline __host__ __device__ int64_t group_tiles(int64_t ntiles) { return ntiles <= (1 << 16) ? 512 : 2048; }
// ... and the most groups that any number of tiles up to ntiles has
inline int64_t most_groups(int64_t ntiles) {
  if (ntiles <= NT_DIRECT_TILES) return 0;
  const int64_t n = (ntiles + group_tiles(ntiles) - 1) / group_tiles(ntiles), small = (1 << 16) / 512;
  return ntiles > (1 << 16) && n < small ? small : n;
}
#define NT_WS_HEADER 32        // doubles in front of the tile partials: a record of the step that wrote them
#define NT_WS_COUNTER 16       // ... and behind it, at this double, the counter of k_reduce_end
#define NT_WS_MAGIC 0x4e54574f524b5350ll

// Scratch of normtest_step_static: the per-tile partial sums and the record of the step, for callers that
// cannot hand over (or allocate) a workspace.  One copy per GPU, held until the process ends.
#define NT_SCRATCH_BYTES (16u << 20)
static __device__ __align__(256) unsigned char scratch[NT_SCRATCH_BYTES];

// Counters with which the blocks of a launch find out which of them comes last (tile_reduce): one, and NT_LEAVES more, each in an
// array of its own so that their counting does not meet.  Zero when the library is loaded, and every launch leaves the ones it was
// given at zero.  A stream has its own (stream_slot), as launches on one stream never run at the same time; taken in turn by all
// streams, a launch that waited on one of them while the others went once round could meet a later call at its counters.
#define NT_STREAMS 4096
static __device__ uint32_t tickets[(1 + NT_LEAVES) * NT_STREAMS];

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

enum { MODE_FULL = 0, MODE_STATS = 1, MODE_ADAMW = 2 };

// One vector access per lane whatever the alignment: gfx950 serves global loads and stores of 8 and 16 bytes from any
// element's address, so the types below promise the compiler no more than that (2 bytes for a pair of bfloat16 words,
// 4 for fp32) and it still emits one dwordx2 / dwordx4.  Rows of an odd-sized matrix without padding (row j starts
// j*d elements in) therefore run like aligned ones: a wave touches one more line per access.  J = 8 bf16,
// d = 30,000,001, unpadded: 224 us (5.4 TB/s) against 406 us (3.0) element by element, which is how such calls ran.
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x3_words __attribute__((ext_vector_type(3), aligned(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// Every array the kernels touch is in global memory; saying so keeps the accesses global (not flat) where the compiler
// cannot trace a pointer back to a kernel argument.
#define NT_GLOBAL __attribute__((address_space(1)))

template <class T, class P>
__device__ inline T ld_nt(P p) {
  return __builtin_nontemporal_load((const T NT_GLOBAL*)p);
}

struct F32 {
  static constexpr int VEC = 4;
  static constexpr int ESIZE = 4;
  typedef u32x4 raw_t;
  __device__ static inline raw_t ldraw(const char NT_GLOBAL* p) { return ld_nt<u32x4_any>(p); }
  // the first n < VEC values, zeros behind them
  __device__ static inline raw_t ldraw_part(const char NT_GLOBAL* p, int n) {
    const uint32_t NT_GLOBAL* q = (const uint32_t NT_GLOBAL*)p;
    raw_t r = {0u, 0u, 0u, 0u};
    if (n > 0) r[0] = q[0];
    if (n > 1) r[1] = q[1];
    if (n > 2) r[2] = q[2];
    return r;
  }
  // coordinates sh, sh+1, ... of the four, zeros behind them
  __device__ static inline raw_t moved(const raw_t& r, int sh) {
    const raw_t x = sh & 1 ? raw_t{r[1], r[2], r[3], 0u} : r, y = sh & 2 ? raw_t{x[2], x[3], 0u, 0u} : x;
    return sh < 4 ? y : raw_t{0u, 0u, 0u, 0u};
  }
  __device__ static inline float val(const raw_t& r, int e) { return __builtin_bit_cast(float, (uint32_t)r[e]); }
  __device__ static inline float ld(const void* base, int64_t i) { return ((const float*)base)[i]; }
};

struct BF16 {
  static constexpr int VEC = 4;
  static constexpr int ESIZE = 2;
  typedef u32x2 raw_t;
  __device__ static inline raw_t ldraw(const char NT_GLOBAL* p) { return ld_nt<u32x2_any>(p); }
  __device__ static inline raw_t ldraw_part(const char NT_GLOBAL* p, int n) {
    const uint16_t NT_GLOBAL* q = (const uint16_t NT_GLOBAL*)p;
    raw_t r = {0u, 0u};
    if (n > 0) r[0] = q[0];
    if (n > 1) r[0] |= (uint32_t)q[1] << 16;
    if (n > 2) r[1] = q[2];
    return r;
  }
  // coordinates sh, sh+1, ... of the four, zeros behind them
  __device__ static inline raw_t moved(const raw_t& r, int sh) {
    const uint64_t x = __builtin_bit_cast(uint64_t, r) >> (16 * sh & 63);
    return __builtin_bit_cast(raw_t, sh < 4 ? x : 0);
  }
  // bfloat16 is the high half of a binary32: widening is a shift or a mask
  __device__ static inline float val(const raw_t& r, int e) {
    uint32_t u = r[e >> 1];
    return __builtin_bit_cast(float, (e & 1) ? (u & 0xffff0000u) : (u << 16));
  }
  __device__ static inline float ld(const void* base, int64_t i) {
    return __builtin_bit_cast(float, (uint32_t)((const uint16_t*)base)[i] << 16);
  }
};

struct StepParams {
  const void* grads; // row 0 of a strided matrix, or (TABLE kernels) a device array of J row pointers
  int64_t ld;       // row stride in elements
  int64_t d;
  int J;
  float* w;
  float* m;
  float* v;
  float* gbar;      // nullptr unless requested
  double* partials; // NT_NV doubles per tile
  double inv_J;
  float beta1, omb1, beta2, omb2; // omb = 1 - beta
  float decay;                    // 1 - lr * weight_decay
  float step_size;                // lr / (1 - beta1^k)
  float inv_sqrt_bc2;             // 1 / sqrt(1 - beta2^k)
  float eps;
  float coord_thr;   // eta^2 b_k (J - ddof) when the coordinate-wise count is wanted, else negative
};

// Start of gradient row j: base + j*ld elements, or the j-th entry of the caller's pointer table.
template <class GT, bool TABLE>
__device__ inline const char* row_base(const StepParams& p, int j) {
  if constexpr (TABLE)   // constant address space: nothing writes the table while the step runs, so scalar loads serve
    return ((const char* const __attribute__((address_space(4)))*)(uintptr_t)p.grads)[j];
  else
    return (const char*)p.grads + (int64_t)j * p.ld * GT::ESIZE;
}

template <class P>
__device__ inline u32x4 ld16(P p) {
  return ld_nt<u32x4_any>(p);
}
template <class P>
__device__ inline void st16(P p, f32x4 x) {
  __builtin_nontemporal_store(x, (f32x4_any NT_GLOBAL*)p);
}

// AdamW on one coordinate (Alg. 1): moments, bias corrections folded into step_size and
// inv_sqrt_bc2, decoupled decay.  sqrt and reciprocal are the 1-ulp hardware forms: the term they
// feed is scaled by lr before it meets w.  The hardware square root flushes subnormal arguments to
// zero, so a second moment below 2^-96 is scaled by 2^64 first (same bits for every normal v).
__device__ inline void adamw_coord(const StepParams& p, float g, float& w, float& m, float& v) {
  m = __builtin_fmaf(p.beta1, m, p.omb1 * g);
  v = __builtin_fmaf(p.beta2, v, (p.omb2 * g) * g);
  const bool tiny = v < 0x1p-96f;
  float root = __builtin_amdgcn_sqrtf(tiny ? v * 0x1p+64f : v);
  root = tiny ? root * 0x1p-32f : root;
  float denom = __builtin_fmaf(root, p.inv_sqrt_bc2, p.eps);
  float upd = (p.step_size * m) * __builtin_amdgcn_rcpf(denom);
  w = __builtin_fmaf(p.decay, w, -upd);
}

// fixed-order sum of a lane's VEC per-coordinate terms
template <int N>
__device__ inline float lane_tree(const float* x) {
  static_assert(N == 4, "per-coordinate terms leave fp32 in groups of four");
  return (x[0] + x[1]) + (x[2] + x[3]);
}

// ---------------------------------------------------------------------------------------------
// Sums over the 64 lanes of a wave, on the vector unit: lanes exchange values by swapping register halves (32 and 16 lanes
// apart) and by row moves (8, 4, 2, 1 apart), not through LDS.  Four sums are formed together: a swap of two values' halves
// leaves each value's lanes in one half of the wave, so the steps below it serve both, and from the third step on all four.
// The additions are those of a butterfly 32, 16, 8, 4, 2, 1 of each value alone.  A tile's five values took 54
// permutes through LDS in every wave of a block, a chain that nothing else covers in a step that lives for a few tiles, and
// where a CU holds one block of 1024 threads: fused step of 4 fp32 rows 10.4 -> 8.5 us at d = 5000 and 13.1 -> 10.5 at 2^20, of
// 8 bf16 rows 129 -> 122 us at 2^24 and 830 -> 820 at 124M, 4 rows with gbar 47.8 -> 41.1 us at 2^24, all launches of a step.
// ---------------------------------------------------------------------------------------------
template <class T>
struct Words {   // a float or double as 32-bit registers
  static constexpr int N = sizeof(T) / 4;
  uint32_t w[N];
};
// lanes 32..63 of x change places with lanes 0..31 of y
template <class T>
__device__ inline void swap_halves(T& x, T& y) {
  Words<T> a = __builtin_bit_cast(Words<T>, x), b = __builtin_bit_cast(Words<T>, y);
#pragma unroll
  for (int k = 0; k < Words<T>::N; ++k) {
    const auto r = __builtin_amdgcn_permlane32_swap(a.w[k], b.w[k], false, false);
    a.w[k] = r[0];
    b.w[k] = r[1];
  }
  x = __builtin_bit_cast(T, a);
  y = __builtin_bit_cast(T, b);
}
// in each half of the wave, lanes 16..31 of x change places with lanes 0..15 of y
template <class T>
__device__ inline void swap_rows(T& x, T& y) {
  Words<T> a = __builtin_bit_cast(Words<T>, x), b = __builtin_bit_cast(Words<T>, y);
#pragma unroll
  for (int k = 0; k < Words<T>::N; ++k) {
    const auto r = __builtin_amdgcn_permlane16_swap(a.w[k], b.w[k], false, false);
    a.w[k] = r[0];
    b.w[k] = r[1];
  }
  x = __builtin_bit_cast(T, a);
  y = __builtin_bit_cast(T, b);
}
// x of the lane OFF further on in the row of 16 lanes (zero past its end)
template <int OFF, class T>
__device__ inline T ahead(T x) {
  Words<T> a = __builtin_bit_cast(Words<T>, x);
#pragma unroll
  for (int k = 0; k < Words<T>::N; ++k) a.w[k] = __builtin_amdgcn_mov_dpp(a.w[k], 0x100 + OFF, 0xf, 0xf, true);
  return __builtin_bit_cast(T, a);
}
// Totals of a, b, c, n over the wave, in the first lane of the first, third, second and fourth row of 16 lanes (lane_value).
// ADD(x, y): x from the lower lanes.
template <class T, class ADD>
__device__ inline T wave_sum4(T a, T b, T c, T n, ADD add) {
  swap_halves(a, b);
  swap_halves(c, n);
  T x = add(a, b), y = add(c, n);   // a in the lower half of x, b in the upper; c and n in y
  swap_rows(x, y);
  x = add(x, y);
  x = add(x, ahead<8>(x));
  x = add(x, ahead<4>(x));
  x = add(x, ahead<2>(x));
  return add(x, ahead<1>(x));
}
// which of the four totals the first lane of a row holds
__device__ inline int lane_value(int lane) { return (lane >> 5) | (lane >> 3 & 2); }
// largest x of the wave (x >= 0), in lane 0
template <class T>
__device__ inline T wave_max(T x) {
  T y = x;
  swap_halves(x, y);
  y = x = __builtin_elementwise_max(x, y);
  swap_rows(x, y);
  x = __builtin_elementwise_max(x, y);
  x = __builtin_elementwise_max(x, ahead<8>(x));
  x = __builtin_elementwise_max(x, ahead<4>(x));
  x = __builtin_elementwise_max(x, ahead<2>(x));
  return __builtin_elementwise_max(x, ahead<1>(x));
}

// ---------------------------------------------------------------------------------------------
// Double-double helpers (error-free transformations; the file is compiled with contraction off).
// ---------------------------------------------------------------------------------------------
struct dd {
  double hi, lo;
};
__host__ __device__ inline dd dd_add(dd x, dd y) {
  double s = x.hi + y.hi;
  double bb = s - x.hi;
  double e = (x.hi - (s - bb)) + (y.hi - bb);
  e += x.lo + y.lo;
  dd r;
  r.hi = s + e;
  r.lo = e - (r.hi - s);
  return r;
}

struct DecideParams {
  int64_t J;
  double eta;
  double max_norm;  // gradient-norm bound of the clipped variant, <= 0: none
  int64_t b_k, b_max, round_to;
  int32_t ddof;
  uint32_t flags;
};

// Record of the step whose tile partials sit in a workspace, kept in its first NT_WS_HEADER doubles so that
// normtest_layer_stats can regroup them per layer and can tell when they belong to another call.
struct WsHeader {
  int64_t magic;
  int64_t tile_coords, ntiles, ngroups;  // ngroups > 0: double-double group partials follow the tile partials
  int64_t d, J;
  int32_t gdtype, has_stats;
  double coord_thr;                      // threshold factor of the coordinate-wise count, negative if off
  DecideParams q;
};
static_assert(sizeof(WsHeader) <= NT_WS_COUNTER * sizeof(double) && sizeof(WsHeader) % 8 == 0, "workspace header");
// The record as words, the form in which kernels take and store it: a struct copied whole goes through scratch memory,
// which every wave of the launch then pays for (fused step -33 %).
struct WsRecord {
  uint64_t word[sizeof(WsHeader) / 8];
};

// Global-norm clipping factor (training specifications of Sec. 5; usual convention with the 1e-6 guard).
__host__ __device__ inline double clip_coef(double gbar_sq, double max_norm) {
  if (!(max_norm > 0.0)) return 1.0;
  const double c = max_norm / (sqrt(gbar_sq) + 1e-6);
  return c < 1.0 ? c : 1.0;
}

// From the sums in r->A, r->B, r->C to ||gbar||^2, ||Var||_1, T, pass and next_b (Alg. 1: test
// statistic, strict comparison with b_k, ceiling, rounding through micro-batch, minibatch and
// global batch, which composes to the next multiple of J*M; Sec. 5: cap at the maximum batch size).
__host__ __device__ inline void decide(const DecideParams& q, nt_result* r) {
  const double Jd = (double)q.J;
  const int64_t cap = (q.b_max > q.b_k) ? q.b_max : q.b_k;
  r->pass = 1;
  r->next_b = q.b_k;
  r->gbar_sq = r->B / (Jd * Jd);
  r->var_l1 = r->C / (double)(q.J - q.ddof);
  r->clip_coef = clip_coef(r->gbar_sq, q.max_norm);
  if (!(__builtin_isfinite(r->A) && __builtin_isfinite(r->B) && __builtin_isfinite(r->C))) {
    r->status |= NT_STATUS_NONFINITE;
    r->T = __builtin_nan("");
    return;
  }
  if (r->gbar_sq == 0.0) {
    r->status |= NT_STATUS_ZERO_GRAD_NORM;
    if (r->C == 0.0) {
      r->T = __builtin_nan("");
    } else {
      r->T = __builtin_inf();
      r->pass = 0;
      r->next_b = cap;
    }
    return;
  }
  const double T = r->var_l1 / (q.eta * q.eta * r->gbar_sq);
  r->T = T;
  if (T > (double)q.b_k) {
    r->pass = 0;
    if (!(T < 4611686018427387904.0)) {
      r->status |= NT_STATUS_T_SATURATED;
      r->next_b = cap;
      return;
    }
    // t < 2^62 and round_to <= 2^31 (validated), so the next multiple fits an int64
    const int64_t t = (int64_t)ceil(T);
    int64_t nb = (t / q.round_to + (t % q.round_to != 0)) * q.round_to;
    if (q.b_max > 0 && nb > q.b_max) {
      nb = q.b_max;
      r->status |= NT_STATUS_CLAMPED;
    }
    r->next_b = nb < q.b_k ? q.b_k : nb;
  }
}

// Running totals of partial records: the NT_NSUM sums in double-double and the largest ratio.
struct Totals {
  dd s[NT_NSUM];
  double mx;
};
__device__ inline void totals_clear(Totals& t) {
#pragma unroll
  for (int k = 0; k < NT_NSUM; ++k) t.s[k] = {0.0, 0.0};
  t.mx = 0.0;
}

// Adds this thread's share (entries threadIdx.x, threadIdx.x + THREADS, ...) of n records into acc.
// PACKED = false: tile partials {A, B, C, n_fail, r_max}; PACKED = true: group partials
// {A, A_lo, B, B_lo, C, C_lo, n, n_lo, r_max, unused}.  Tile partials are loaded up to eight rounds
// at a time: one round after the other, 2048 records in a block of 256 threads wait for memory eight times (groups of 2048
// 7.2 -> 4.5 us).  Group partials are few (one per 1M coordinates or more, up to 2^19 tiles at most 256, one round), so theirs are
// not.  What lies past the end reads as the
// last record and counts as zeros, which change nothing.
template <int THREADS, bool PACKED>
__device__ inline void totals_accumulate(const double* in, int64_t n, Totals& acc) {
  constexpr int BATCH = PACKED ? 1 : THREADS <= 256 ? 8 : 4;
  constexpr int LEN = PACKED ? 2 * NT_NV : NT_NV, USED = PACKED ? 2 * NT_NSUM + 1 : NT_NV;
  for (int64_t t0 = 0; t0 < n; t0 += BATCH * THREADS) {
    double rec[BATCH][USED];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int64_t t = t0 + b * THREADS + threadIdx.x;
      if (t0 + b * THREADS < n) {
#pragma unroll
        for (int k = 0; k < USED; ++k) rec[b][k] = in[LEN * (t < n ? t : n - 1) + k];
      }
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      if (t0 + b * THREADS < n) {
        const bool there = t0 + b * THREADS + threadIdx.x < n;
#pragma unroll
        for (int k = 0; k < NT_NSUM; ++k) {
          const dd x = PACKED ? dd{rec[b][2 * k], rec[b][(2 * k + 1) % USED]} : dd{rec[b][k], 0.0};
          acc.s[k] = dd_add(acc.s[k], there ? x : dd{0.0, 0.0});
        }
        acc.mx = __builtin_fmax(acc.mx, rec[b][USED - 1]);
      }
    }
  }
}

// Total of the accumulators of the block's first THREADS threads (whole waves); all threads of the block take part, thread 0
// returns the totals.
template <int THREADS>
__device__ inline void block_totals_finish(Totals& acc, double (*sh)[2 * NT_NV], Totals& tot) {
  static_assert(NT_NSUM == 4, "wave_sum4");
  const dd x = wave_sum4(acc.s[0], acc.s[1], acc.s[2], acc.s[3], [](dd p, dd q) { return dd_add(p, q); });
  const double mx = wave_max(acc.mx);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave < THREADS / 64 && (lane & 15) == 0) {
    sh[wave][2 * lane_value(lane)] = x.hi;
    sh[wave][2 * lane_value(lane) + 1] = x.lo;
    if (lane == 0) sh[wave][2 * NT_NSUM] = mx;
  }
  __syncthreads();
  if (wave == 0) {
    // the sums of the waves in their order, one of the four per lane, then all to thread 0
    const int k = lane < NT_NSUM ? lane : 0;
    dd t = {sh[0][2 * k], sh[0][2 * k + 1]};
    double m = sh[0][2 * NT_NSUM];
#pragma unroll
    for (int wv = 1; wv < THREADS / 64; ++wv) {
      t = dd_add(t, dd{sh[wv][2 * k], sh[wv][2 * k + 1]});
      m = __builtin_fmax(m, sh[wv][2 * NT_NSUM]);
    }
    tot.s[0] = t;
    tot.s[1] = ahead<1>(t);
    tot.s[2] = ahead<2>(t);
    tot.s[3] = ahead<3>(t);
    tot.mx = m;
  }
}

// Sum of n records (layouts as in totals_accumulate) by the block's first THREADS threads, in an order that does not depend on
// the block's size; thread 0 returns the totals.
template <int THREADS, bool PACKED>
__device__ inline void block_totals(const double* in, int64_t n, double (*sh)[2 * NT_NV], Totals& tot) {
  Totals acc;
  totals_clear(acc);
  if (threadIdx.x < THREADS) totals_accumulate<THREADS, PACKED>(in, n, acc);
  block_totals_finish<THREADS>(acc, sh, tot);
}

// From the totals of a step to the record of it in the workspace and the caller's result; one thread.
__device__ inline void write_record(const Totals& tot, const DecideParams& q, nt_result* out, const WsRecord& hdr,
                                    WsRecord* hdr_out) {
  const bool stats = (q.flags & NT_DO_STATS) != 0;
#pragma unroll
  for (size_t k = 0; k < sizeof(WsHeader) / 8; ++k) hdr_out->word[k] = hdr.word[k];
  nt_result r;
  r.status = 0;
  const bool coord = stats && (q.flags & NT_COORD_TEST);
  r.coord_fail = coord ? (int64_t)tot.s[3].hi : -1;
  r.coord_max_ratio = coord ? tot.mx : -1.0;
  const double nan = __builtin_nan("");
  if (!stats) {
    r.A = r.B = r.C = r.A_lo = r.B_lo = r.C_lo = nan;
    r.gbar_sq = r.var_l1 = r.T = nan;
    r.clip_coef = 1.0;
    r.pass = 1;
    r.next_b = q.b_k;
    r.status = NT_STATUS_NO_STATS;
  } else {
    r.A = tot.s[0].hi; r.A_lo = tot.s[0].lo;
    r.B = tot.s[1].hi; r.B_lo = tot.s[1].lo;
    r.C = tot.s[2].hi; r.C_lo = tot.s[2].lo;
    if (q.flags & NT_PARTIAL) {
      r.gbar_sq = r.var_l1 = r.T = nan;
      r.clip_coef = 1.0;
      r.pass = 1;
      r.next_b = q.b_k;
      r.status = NT_STATUS_PARTIAL_ONLY;
      if (!(__builtin_isfinite(r.A) && __builtin_isfinite(r.B) && __builtin_isfinite(r.C)))
        r.status |= NT_STATUS_NONFINITE;
    } else {
      decide(q, &r);
    }
  }
  *out = r;
}

// What a step takes along whose own kernel writes the result.
struct Finish {
  DecideParams q;
  WsRecord hdr;
  WsRecord* hdr_out;
  nt_result* out;     // null: k_finalize follows
  uint32_t* ticket;   // steps of more than one tile: where its blocks count themselves
};
// The counter of one block of such a step: its leaf (blocks of neighbouring numbers have different ones), or the only one.
__device__ inline uint32_t* leaf_of(uint32_t* ticket, int64_t ntiles) {
  return ticket && ntiles > NT_LEAF_TILES ? ticket + (1 + blockIdx.x % NT_LEAVES) * NT_STREAMS : ticket;
}
__device__ inline uint32_t count_up(uint32_t* ticket) {
  return __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Whether the block that found `before` others at its counter is the last of the step's: it may then read what all of them have
// written, and the counters are as they were given.  They are put back behind the acquire, which waits for the stores
// before it: in front, a trip to memory more (fused step of 4 fp32 rows 7.11 -> 6.88 us at d = 5000, 9.12 -> 8.87 at 2^20; of 64 bf16
// rows 9.54 -> 9.38 and, at 2^18, 11.83 -> 11.46).
__device__ inline bool last_block(uint32_t* ticket, uint32_t ntiles, uint32_t before) {
  uint32_t* const leaf = leaf_of(ticket, ntiles);
  uint32_t all = ntiles;
  if (ntiles > NT_LEAF_TILES) {
    if (before != (ntiles - blockIdx.x % NT_LEAVES + NT_LEAVES - 1) / NT_LEAVES - 1) return false;
    before = count_up(ticket);
    all = NT_LEAVES;
  }
  const bool last = before == all - 1;
  if (last) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (leaf != ticket) __hip_atomic_store(leaf, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return last;
}

// ---------------------------------------------------------------------------------------------
// The parts of a tile's work.
// ---------------------------------------------------------------------------------------------
// What a lane gathers over the sweeps of one tile: the three sums in fp64 (each fed with fp32 sums of four
// coordinates), the number of coordinates failing the coordinate-wise test and their largest ratio.
struct LaneAcc {
  double A = 0.0, B = 0.0, C = 0.0;
  int nfail = 0;
  float rmax = 0.f;
};

// What the first wave of a block keeps of its tile's end in a step that writes its own result: its lane's value of the tile
// partial and, in lane 0, how many blocks had counted themselves before.
struct TileEnd {
  double value;
  uint32_t before;
};

// Block partial of one tile -> partials[NT_NV*tile ..].
// END: the launch has a block per tile and its last one adds up the partials (k_step_end).  The partial then goes through this
// XCD's L2 to memory, and once it is there the block counts itself.  Both accesses are relaxed on purpose: a release would
// write back all of the L2, in every block.  What orders them is the machine, not the language: on gfx950 a store of agent scope is
// written through (sc1), s_waitcnt vmcnt(0) returns once it has reached the memory that all XCDs share, and the count is issued by
// the same wave behind it; the last block's acquire then drops what its own caches may hold of the partials.  Nobody waits for another
// block; the state, if any, is stored after the counting, so that its way to memory is not waited for.
template <int BLOCK, bool END>
__device__ inline TileEnd tile_reduce(const LaneAcc& acc, double (*red)[NT_NV], double* partials,
                                      int64_t tile, uint32_t* ticket) {
  const double x = wave_sum4(acc.A, acc.B, acc.C, (double)acc.nfail, [](double p, double q) { return p + q; });
  const float r = wave_max(acc.rmax);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if ((lane & 15) == 0) {
    red[wave][lane_value(lane)] = x;
    if (lane == 0) red[wave][NT_NSUM] = (double)r;
  }
  __syncthreads();
  TileEnd end = {0.0, 0};
  if (threadIdx.x < NT_NV) {
    // the waves in their order, one of the five values per lane
    double t = red[0][threadIdx.x];
#pragma unroll
    for (int wv = 1; wv < BLOCK / 64; ++wv) {
      const double y = red[wv][threadIdx.x];
      t = threadIdx.x < NT_NSUM ? t + y : __builtin_fmax(t, y);
    }
    double* const to = partials + NT_NV * tile + threadIdx.x;
    if constexpr (END) {
      end.value = t;
      __hip_atomic_store(to, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (ticket) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (threadIdx.x == 0) end.before = count_up(ticket);
      }
    } else {
      *to = t;
      // the counter of the reduction that may follow, which is a kernel of its own
      if (tile == 0 && threadIdx.x == 0) *(uint32_t*)(partials - NT_WS_HEADER + NT_WS_COUNTER) = 0;
    }
  }
  return end;
}

// Coordinate-wise form of the test (Sec. 4, Prop. 1): with thr = eta^2 b_k (J - ddof), a coordinate with centred
// sum c and mean gb has the ratio c / (thr gb^2) and fails when that exceeds one.  A coordinate without spread
// has ratio 0 whatever its mean; spread around a zero mean gives +inf.  thr < 0 switches both off.
__device__ inline void coord_test(float thr, float c, float gb, LaneAcc& acc) {
  if (thr >= 0.f) {
    const float den = thr * (gb * gb);
    acc.nfail += (c > den) ? 1 : 0;
    const float rho = (c == 0.f) ? 0.f : c / den;
    acc.rmax = __builtin_fmaxf(acc.rmax, rho);
  }
}

// Per-chunk bookkeeping of the walk of more than 16 fp32 rows (walk_shifted).  For one coordinate and a chunk of nb rows with shift
// K (the running mean before the chunk, or the first row for the first chunk) two sums have been accumulated:
// sb = sum x in fp64 (exact for all practical purposes, so the mean handed to AdamW is correctly rounded
// even when the rows cancel) and q = sum (x - K)^2 in fp32.  With sr = sb - nb K, the sum of the shifted values,
//   chunk centred sum   M2_b = q - sr^2/nb
//   chunk sum of squares  a_b = q + K (2 sr + nb K)
// and the chunk is merged into the running (S, M2) with  S += sb,  M2 += M2_b + delta^2 na nb/(na + nb),
// delta = mean_b - mean_a.  Returns the shift for the next chunk.
// inv_na, inv_n: 1/na and 1/(na + nb).
__device__ inline float chunk_merge(bool first, int na, int nb, double inv_na, double inv_n, float K, double sb, float q,
                                    double& S, float& M2, float& a) {
  const double sr = __builtin_fma(-(double)K, (double)nb, sb);
  const float srf = (float)sr;
  const float nbf = (float)nb;
  const double inv_nb = 1.0 / (double)nb;
  const float M2b = __builtin_fmaf(-(srf * (float)inv_nb), srf, q);
  a += __builtin_fmaf(K, __builtin_fmaf(nbf, K, 2.0f * srf), q);
  if (first) {
    S = sb;
    M2 = M2b;
  } else {
    const float coef = ((float)na * nbf) / (float)(na + nb);
    const float delta = (float)(((double)K - S * inv_na) + sr * inv_nb);
    M2 = M2 + __builtin_fmaf(delta * delta, coef, M2b);
    S = S + sb;
  }
  return (float)(S * inv_n);
}

// More than 16 bf16 rows: sum x and sum x^2 of a coordinate in fp64, hence the centred sum without a shift.  x^2 has 16 bits, so both
// sums are exact unless the rows' magnitudes lie a factor of 2^14 or more apart, where no centred sum is small.  Against 64 bits C is
// 2.4e-10 off (128 rows, d = 1,000,003) and 2.2e-9 (24 rows, 100,003), where sums of fp32 squares with a shift were 3.4e-9 and 1.6e-8.
// An element takes 17 cycles of a SIMD, with the shift and the merges 27.  Less arithmetic also sends a block's loads in denser bursts, which
// at some lengths makes the short tiles of 2048 coordinates slower.  Shifted -> by moments in those tiles, us: fused step of 20 / 48 rows at
// d = 2^21 25.8 / 50.2 -> 26.8 / 52.2, of 40 at 5e6 92.6 -> 95.1, but of 20 at 2.5e6 33.9 -> 30.7; statistics of 20 / 100 rows at 1e7
// 66.7 / 306 -> 64.5 / 300.  The rows are added up in up to four segments of whole chunks, one after the other within a segment, and
// the segments in their order: the waves of a block can then take one each (tile_split) with the same bits.
__host__ __device__ inline int segment_rows(int J) {
  return ((J + NT_MCHUNK - 1) / NT_MCHUNK + NT_SEGMENTS - 1) / NT_SEGMENTS * NT_MCHUNK;
}
// sum x^2 - S^2 / J: the difference J Q - S^2 with the product's rounding error, so that equal rows give zero
__device__ inline float centred(int J, double inv_J, double S, double Q) {
  const double n = (double)J, t = n * Q;
  const double c = __builtin_fma(-S, S, t) + __builtin_fma(n, Q, -t);
  return (float)((c < 0.0 ? 0.0 : c) * inv_J);
}

// ---------------------------------------------------------------------------------------------
// One coordinate by itself, up to NT_JCHUNK rows and any alignment: what the per-layer table needs at a layer's ends, where a layer
// covers a part of a tile (piece_sums).  The operations on a coordinate are those of the tiles below, in their order, and have to
// stay so; only the sums over coordinates are formed in another order.  The J loads of a coordinate are issued together.
// ---------------------------------------------------------------------------------------------
template <class GT, bool TABLE, int J_T>
__device__ inline void coord_stats(const StepParams& p, int64_t i, double& S, float& M2, float& a) {
  float x[J_T];
#pragma unroll
  for (int j = 0; j < J_T; ++j) x[j] = GT::ld(row_base<GT, TABLE>(p, j), i);
  S = (double)x[0];
#pragma unroll
  for (int j = 1; j < J_T; ++j) S += (double)x[j];
  const float mb = (float)(S * p.inv_J);
  M2 = 0.f;
  a = 0.f;
#pragma unroll
  for (int j = 0; j < J_T; ++j) {
    const float r = x[j] - mb;
    M2 = __builtin_fmaf(r, r, M2);
    a = __builtin_fmaf(x[j], x[j], a);
  }
}

// ---------------------------------------------------------------------------------------------
// Loads and stores of a lane's VEC coordinates i0 .. i0+3.  part: the tile may reach past d.  A group that does is loaded by the
// same instruction as every other, as the vector's last four coordinates, and where there are sums moved down to where it belongs
// (Reach, settle); what lies past d is then zero rows on zero state, which add exact zeros to every sum.  Its 1 to 3 values are
// stored one by one.  The arithmetic is the same for whole and part tiles, hence the same bits.  Element by element, in a branch of its own,
// such a group's rows were a chain of loads that a short vector waits for (d = 100,003: fused step of 16 bf16 rows 11.1 -> 9.9
// us, of 512 rows 126 -> 106, statistics of 64 / 256 rows in tables 29.6 -> 15.2 and 119 -> 56).
// ---------------------------------------------------------------------------------------------
// coordinates i0 .. i0+3 that lie below d: 4 or fewer, 0 or negative where none does
__device__ inline int below(int64_t d, int64_t i0) { return (int)(d - i0 < 4 ? (d - i0 < 0 ? 0 : d - i0) : 4); }
// Where a lane's four coordinates start: s0, the sweep's first coordinate (the same for the whole block), plus the lane's
// own offset.  scalar() pins a block-uniform address to scalar registers: every access is then a scalar base and one
// shared lane offset, where the compiler would otherwise form a 64-bit vector address per row and array (fused step at 8
// rows: 79 vector registers instead of 88; 4 rows in tables, d = 304.6M: 1737 -> 1684 us).
struct Place {
  int64_t s0;
  uint32_t u;
  __device__ inline int64_t i0() const { return s0 + u; }
};
template <class T>
__device__ inline T NT_GLOBAL* scalar(T* p) {
  const uint64_t a = (uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)a), hi = __builtin_amdgcn_readfirstlane((int)(a >> 32));
  return (T NT_GLOBAL*)(((uint64_t)hi << 32) | lo);
}
template <class T>
__device__ inline T NT_GLOBAL* at(T* base, const Place& pl) {
  return scalar(base + pl.s0) + pl.u;
}

// Where a lane's vector loads start, at coordinate s0 + u (s0 uniform), and by how many coordinates sh what they return has to be
// moved: in a part tile the group that reaches past d, and every group behind it, loads the vector's last four coordinates
// instead.  What it reads of its neighbour's coordinates, which that lane may have updated by then, is moved out.  A vector of
// fewer than four has no such place; its values are loaded one by one (load_sweep).
struct Reach {
  int64_t s0;
  uint32_t u;
  int sh;
};
__device__ inline Reach reach(bool part, const StepParams& p, const Place& pl) {
  if (__builtin_expect(!part || p.d < 4, 1)) return {pl.s0, pl.u, 0};
  // as far from s0 - 4 as from s0 - 1 on the last four coordinates begin, so that lanes' offsets stay positive
  const int64_t s0 = pl.s0 < 4 ? 0 : pl.s0 - 4;
  const int64_t last = p.d - 4 - s0;
  const uint32_t want = (uint32_t)(pl.s0 - s0) + pl.u;
  const uint32_t most = last < (1 << 20) ? (uint32_t)last : 1u << 20;
  const uint32_t u = want < most ? want : most;
  return {s0, u, (int)(want - u)};
}
// The copies of the code of a tile.  AdamW only of at most 16 rows has one, in which part tiles differ by branches that are the same
// for the whole block, and so has the class for long vectors beyond 20 bf16 rows, whose generations stay in step better (32 rows,
// d = 2^24: 245 us against 256).  Elsewhere whole tiles and part tiles have a copy each (with one, the fused step of 4 fp32 rows
// takes 7.4 instead of 6.7 us at d = 5000, of 8 bf16 rows 9843 instead of 9745 at 1.5e9; sweeps of statistics could not overlap); see
// also whole_copy.
template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool DEFER_T>
constexpr bool one_copy() {
  return MODE == MODE_ADAMW && !DEFER_T &&
         (J_T > 0 || (GT::ESIZE == 2 && BLOCK == NT_BLOCK_LARGE && ITERS == NT_ITERS_LARGE));
}
// Whether a part tile's rows and state are moved to the lane's own coordinates once they are loaded.  Sums need that: what lies past
// d has to be zeros.  With AdamW only a lane updates the coordinates that it has loaded, and stores its own ones among them (store4):
// moving the rows is a long way through cold code (16 / 8 fp32 rows, d = 1000: 6.1 / 4.6 us with it, 4.7 / 3.8 without).
// In the classes for long vectors tables keep it, where two copies without it would be given scratch memory.
template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool TABLE, bool DEFER_T>
constexpr bool moves_rows() {
  return MODE != MODE_ADAMW || (J_T == 0 && TABLE && BLOCK * ITERS == NT_BLOCK_LARGE * NT_ITERS_LARGE &&
                                !one_copy<GT, J_T, MODE, BLOCK, ITERS, DEFER_T>());
}
// Rows or state as loaded -> as they belong, if they are moved, and where the lane then is.
template <class GT, int N, bool MOVES>
__device__ inline Reach settle(bool part, const Place& pl, const Reach& r, typename GT::raw_t* raw) {
  if constexpr (!MOVES) return r;
  if (__builtin_expect(part, 0)) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      raw[j] = GT::moved(raw[j], r.sh);
      asm volatile("" : "+v"(raw[j]));   // one row after the other: interleaved, 16 fp32 rows need registers there are not
    }
  }
  return {pl.s0, pl.u, 0};
}

// Rows j0, j0+1, ... at coordinate s0, one after the other: a matrix is walked by adding its row stride.
template <class GT, bool TABLE>
struct RowWalk {
  const StepParams& p;
  int j;
  int64_t off;
  const char* at;
  __device__ inline RowWalk(const StepParams& p_, int j0, int64_t s0)
      : p(p_), j(j0), off(s0 * GT::ESIZE), at(TABLE ? nullptr : row_base<GT, false>(p_, j0) + off) {}
  __device__ inline const char NT_GLOBAL* next() {
    if constexpr (TABLE) return scalar(row_base<GT, true>(p, j++) + off);
    const char NT_GLOBAL* a = scalar(at);
    at = (const char*)(uintptr_t)a + p.ld * GT::ESIZE;
    return a;
  }
};

// Rows j0 .. j0+N-1 of the lane's coordinates, and with STATE w, m, v too, as loaded (see settle).  The sweep's first coordinate
// lies below d.  Every row of a vector of fewer than four coordinates is used at once, so that no load is pending behind that
// branch: the wait before each row's first use would have to allow for it and be a wait for all rows.
template <class GT, bool TABLE, int N, bool STATE>
__device__ inline void load_sweep(bool part, const StepParams& p, int j0, const Reach& r, typename GT::raw_t* raw, u32x4* state) {
  const uint32_t lane = r.u * GT::ESIZE;
  const Place pl = {r.s0, r.u};
  RowWalk<GT, TABLE> row(p, j0, r.s0);
  if (__builtin_expect(!part || p.d >= 4, 1)) {
#pragma unroll
    for (int j = 0; j < N; ++j) raw[j] = GT::ldraw(row.next() + lane);
    if constexpr (STATE) {
      state[0] = ld16(at(p.w, pl));
      state[1] = ld16(at(p.m, pl));
      state[2] = ld16(at(p.v, pl));
    }
  } else {
    const int n = below(p.d, pl.i0());
#pragma unroll
    for (int j = 0; j < N; ++j) {
      raw[j] = GT::ldraw_part(row.next() + lane, n);
      asm volatile("" : "+v"(raw[j]));
    }
    if constexpr (STATE) {
      state[0] = F32::ldraw_part((const char NT_GLOBAL*)at(p.w, pl), n);
      state[1] = F32::ldraw_part((const char NT_GLOBAL*)at(p.m, pl), n);
      state[2] = F32::ldraw_part((const char NT_GLOBAL*)at(p.v, pl), n);
    }
  }
}
template <class GT, bool TABLE, int N>
__device__ inline void load_rows(bool part, const StepParams& p, int j0, const Reach& r, typename GT::raw_t* raw) {
  load_sweep<GT, TABLE, N, false>(part, p, j0, r, raw, nullptr);
}

// Values of the coordinates at r.  Of a group that was loaded from the vector's end and not moved (r.sh > 0), the lane's own ones
// are those from sh on.
__device__ inline void store4(bool part, const StepParams& p, float* base, const Reach& r, f32x4 x) {
  const Place pl = {r.s0, r.u};
  const int n = part ? below(p.d, pl.i0()) : 4;
  if (__builtin_expect(n >= 4 && r.sh == 0, 1)) {
    st16(at(base, pl), x);
  } else {
    float NT_GLOBAL* q = at(base, pl);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e >= r.sh && e < n) q[e] = x[e];
  }
}

// AdamW on VEC coordinates whose state was loaded as 16-byte vectors, then the stores.
__device__ inline void adamw_store(bool part, const StepParams& p, const Reach& r, const float* gb,
                                   const u32x4* state) {
  f32x4 ow, om, ov;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float w = __builtin_bit_cast(float, (uint32_t)state[0][e]);
    float m = __builtin_bit_cast(float, (uint32_t)state[1][e]);
    float v = __builtin_bit_cast(float, (uint32_t)state[2][e]);
    adamw_coord(p, gb[e], w, m, v);
    ow[e] = w;
    om[e] = m;
    ov[e] = v;
  }
  if (__builtin_expect(!part, 1)) {
    const Place pl = {r.s0, r.u};
    st16(at(p.w, pl), ow);
    st16(at(p.m, pl), om);
    st16(at(p.v, pl), ov);
  } else {
    store4(true, p, p.w, r, ow);
    store4(true, p, p.m, r, om);
    store4(true, p, p.v, r, ov);
  }
}

// ---------------------------------------------------------------------------------------------
// Tiles, J <= 16 known at compile time: all J rows of a group of VEC coordinates sit in registers.
// The row sum is carried in fp64 so that the mean is correctly rounded even when the rows cancel.
// ---------------------------------------------------------------------------------------------
// One sweep's arithmetic: the means of the lane's VEC coordinates into gb, the sweep's sums into acc.
template <class GT, int J, int MODE, bool COORD>
__device__ inline void sweep_rows(const StepParams& p, const typename GT::raw_t* raw, float* gb, LaneAcc& acc) {
  constexpr int VEC = GT::VEC;
  double s[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) s[e] = (double)GT::val(raw[0], e);
#pragma unroll
  for (int j = 1; j < J; ++j)
#pragma unroll
    for (int e = 0; e < VEC; ++e) s[e] += (double)GT::val(raw[j], e);
#pragma unroll
  for (int e = 0; e < VEC; ++e) gb[e] = (float)(s[e] * p.inv_J);

  if constexpr (MODE != MODE_ADAMW) {
    float a[VEC], c[VEC], b[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) a[e] = c[e] = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float x = GT::val(raw[j], e);
        const float r = x - gb[e];
        c[e] = __builtin_fmaf(r, r, c[e]);
        a[e] = __builtin_fmaf(x, x, a[e]);
      }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float sf = (float)s[e];
      b[e] = sf * sf;
      if constexpr (COORD) coord_test(p.coord_thr, c[e], gb[e], acc);
    }
    acc.A += (double)lane_tree<VEC>(a);
    acc.B += (double)lane_tree<VEC>(b);
    acc.C += (double)lane_tree<VEC>(c);
  }
}

// Statistics kernels whose loads have to be kept together: at these row counts the compiler sinks the last two or three loads
// of a sweep below the first sums, and every sweep then waits for memory three times (read-only statistics, d = 2^21: 15 bf16
// rows 27.4 -> 21.5 us, 11 / 15 fp32 rows 25.4 -> 23.8 and 35.6 -> 30.3; d = 1e8: 446 -> 434, +-0.3 %).  At the other counts
// it issues them together by itself, and holding it to that only keeps sums from starting early (14 and 16 bf16 rows,
// d = 5e6 .. 1e7: +0.9 .. 2.7 % time).
constexpr bool pin_loads(int esize, int J, bool coord) { return !coord && (J == 15 || (J == 11 && esize == 4)); }

// State update interleaved with the rows: each sweep reads its rows and w, m, v, and writes the state back.
template <class GT, int J, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool COORD, bool PART, bool END>
__device__ inline TileEnd tile_rows(bool part, const StepParams& p, int64_t tile, double (*red)[NT_NV],
                                    uint32_t* ticket) {
  constexpr int VEC = GT::VEC;
  constexpr int TILE = BLOCK * VEC * ITERS;
  constexpr bool EARLY = END && MODE == MODE_FULL;   // the sums are handed on before the state is stored
  static_assert(!EARLY || ITERS == 1, "the sums are complete after the only sweep");
  LaneAcc acc;
  TileEnd end = {0.0, 0};
  // a statistics-only sweep with few rows has little in flight per lane: overlap sweeps up to about 64 bytes (read-only,
  // 128 bytes are 35 % slower at 4 bf16 rows), and where gbar is stored two sweeps of 64 bytes (8 bf16 rows, d = 2e8: 656
  // -> 630 us; 4 fp32 rows 674 -> 650; two sweeps of 40 or 48 bytes are 10 and 4 % slower than one)
  constexpr int ROW_BYTES = VEC * GT::ESIZE;
  constexpr int WANT = (GBAR && J * ROW_BYTES >= 64 ? 128 : 64) / (J * ROW_BYTES);
  constexpr int U = (MODE == MODE_STATS && ITERS > 1 && !PART) ? (WANT >= 4 ? 4 : (WANT >= 2 ? 2 : 1)) : 1;
#pragma unroll U
  for (int it = 0; it < ITERS; ++it) {
    const Place pl = {tile * TILE + (int64_t)it * BLOCK * VEC, threadIdx.x * VEC};
    if (PART && part && pl.s0 >= p.d) break;
    typename GT::raw_t raw[J];
    u32x4 state[3];
    const Reach at = reach(PART && part, p, pl);
    load_sweep<GT, TABLE, J, MODE != MODE_STATS>(PART && part, p, 0, at, raw, state);
    if constexpr (MODE == MODE_STATS && U == 1 && !PART && pin_loads(GT::ESIZE, J, COORD)) __builtin_amdgcn_sched_barrier(0);
    if constexpr (MODE != MODE_STATS) {
      // Every load of the sweep is issued before any arithmetic: the compiler must neither sink loads below
      // the arithmetic that precedes their use nor hoist arithmetic between them (measured: up to 5 % at 16
      // rows against schedules that issue the state loads after the rows have arrived).  Statistics-only
      // tiles are left free so that consecutive sweeps can overlap.
      __builtin_amdgcn_sched_barrier(0);
    }
    const Reach out = settle<GT, J, MODE != MODE_ADAMW>(PART && part, pl, at, raw);
    float gb[VEC];
    sweep_rows<GT, J, MODE, COORD>(p, raw, gb, acc);
    if constexpr (EARLY) end = tile_reduce<BLOCK, true>(acc, red, p.partials, tile, ticket);
    if constexpr (MODE != MODE_STATS) {
      settle<F32, 3, MODE != MODE_ADAMW>(PART && part, pl, at, state);
      adamw_store(PART && part, p, out, gb, state);
    }
    if (GBAR && p.gbar) store4(PART && part, p, p.gbar, out, f32x4{gb[0], gb[1], gb[2], gb[3]});
  }
  if constexpr (MODE != MODE_ADAMW && !EARLY) end = tile_reduce<BLOCK, END>(acc, red, p.partials, tile, ticket);
  // AdamW-only tiles end with a block barrier like the other modes: the waves of a block then finish together
  // and the next block's waves start together (measured +2 %)
  if constexpr (MODE == MODE_ADAMW) __syncthreads();
  return end;
}

template <int MODE, int BLOCK, int ITERS, bool GBAR, bool PART, bool MOVES>
__device__ inline void deferred_sweeps(const StepParams& p, int64_t tile, const f32x4* gbs) {
  constexpr int VEC = 4;
  constexpr int TILE = BLOCK * VEC * ITERS;
#pragma unroll 2
  for (int it = 0; it < ITERS; ++it) {
    const Place pl = {tile * TILE + (int64_t)it * BLOCK * VEC, threadIdx.x * VEC};
    if (PART && pl.s0 >= p.d) break;
    const f32x4 g4 = gbs[it * BLOCK + threadIdx.x];   // this lane's own values: no barrier needed for them
    const float gb[VEC] = {g4[0], g4[1], g4[2], g4[3]};
    Reach out = {pl.s0, pl.u, 0};
    if constexpr (MODE != MODE_STATS) {
      u32x4 state[3];
      const Reach at = reach(PART, p, pl);
      load_sweep<F32, false, 0, true>(PART, p, 0, at, nullptr, state);
      out = settle<F32, 3, MOVES>(PART, pl, at, state);
      adamw_store(PART, p, out, gb, state);
    }
    if (GBAR && p.gbar) store4(PART, p, p.gbar, out, g4);
  }
}

// The end of a tile whose state update was deferred: the means of all its sweeps wait in LDS (gbs) until every
// row has been read, then w, m, v of all sweeps are read and written in one go.  The memory system charges writes
// sprinkled among reads several times their volume; gathered at the end of a block's life, and with all blocks
// of a launch living at the same time (one generation per launch), they reach it as a dense burst.
template <int MODE, int BLOCK, int ITERS, bool GBAR, bool PART, bool END, bool MOVES>
__device__ inline TileEnd deferred_update(const StepParams& p, int64_t tile, double (*red)[NT_NV],
                                          const LaneAcc& acc, const f32x4* gbs, uint32_t* ticket) {
  constexpr int VEC = 4;
  constexpr int TILE = BLOCK * VEC * ITERS;
  // the barrier inside keeps the waves of the block together on their way into the write phase
  TileEnd end = {0.0, 0};
  if constexpr (MODE != MODE_ADAMW)
    end = tile_reduce<BLOCK, END>(acc, red, p.partials, tile, ticket);
  else
    __syncthreads();
  if (MODE != MODE_STATS || p.gbar) {
    // a copy of the loop for whole tiles: its sweeps overlap
    if (!PART || tile * TILE + TILE <= p.d)
      deferred_sweeps<MODE, BLOCK, ITERS, GBAR, false, false>(p, tile, gbs);
    else
      deferred_sweeps<MODE, BLOCK, ITERS, GBAR, true, MOVES>(p, tile, gbs);
  }
  return end;
}

// Deferred state update, rows in registers: the sweeps read rows only.
template <class GT, int J, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool PART>
__device__ inline void tile_defer(const StepParams& p, int64_t tile, double (*red)[NT_NV],
                                       f32x4* gbs) {
  constexpr int VEC = GT::VEC;
  static_assert(VEC == 4, "one 16-byte LDS slot per lane and sweep");
  constexpr int TILE = BLOCK * VEC * ITERS;
  LaneAcc acc;
#pragma unroll NT_DEFER_UNROLL
  for (int it = 0; it < ITERS; ++it) {
    const Place pl = {tile * TILE + (int64_t)it * BLOCK * VEC, threadIdx.x * VEC};
    if (PART && pl.s0 >= p.d) break;
    typename GT::raw_t raw[J];
    const Reach at = reach(PART, p, pl);
    load_rows<GT, TABLE, J>(PART, p, 0, at, raw);
    settle<GT, J, MODE != MODE_ADAMW>(PART, pl, at, raw);
    float gb[VEC];
    sweep_rows<GT, J, MODE, true>(p, raw, gb, acc);
    gbs[it * BLOCK + threadIdx.x] = f32x4{gb[0], gb[1], gb[2], gb[3]};
  }
  deferred_update<MODE, BLOCK, ITERS, GBAR, PART, false, MODE != MODE_ADAMW>(p, tile, red, acc, gbs, nullptr);
}

// ---------------------------------------------------------------------------------------------
// Tile, J > 16: rows are walked NT_MCHUNK at a time.  bf16 rows: one pass over a chunk adds its values and their squares, both in
// fp64 (walk_moments, centred).  fp32 rows: it gives the chunk's plain sum (fp64) and the sum of squares of the values shifted by
// K, the running mean of the rows before it, hence its centred sum of squares without cancellation (walk_shifted, chunk_merge).
// ---------------------------------------------------------------------------------------------
template <class GT, bool MOVES, int N>
__device__ inline void chunk_accumulate(typename GT::raw_t* raw, const Reach& at, const float* K, double* sb, float* q) {
  constexpr int VEC = GT::VEC;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if constexpr (MOVES) raw[j] = GT::moved(raw[j], at.sh);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float x = GT::val(raw[j], e);
      const float r = x - K[e];
      sb[e] += (double)x;
      q[e] = __builtin_fmaf(r, r, q[e]);
    }
  }
}
template <int VEC>
__device__ inline void chunk_clear(double* sb, float* q) {
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    sb[e] = 0.0;
    q[e] = 0.f;
  }
}

template <class GT, bool MOVES, int N>
__device__ inline void chunk_moments(typename GT::raw_t* raw, const Reach& at, double* s, double* q) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if constexpr (MOVES) raw[j] = GT::moved(raw[j], at.sh);
#pragma unroll
    for (int e = 0; e < GT::VEC; ++e) {
      const double x = (double)GT::val(raw[j], e);
      s[e] += x;
      q[e] = __builtin_fma(x, x, q[e]);
    }
  }
}
template <int VEC>
__device__ inline void segment_end(double* S, double* Q, double* s, double* q) {
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    S[e] += s[e];
    Q[e] += q[e];
    s[e] = q[e] = 0.0;
  }
}
// The last nb < 16 rows, in runs of 8, 4, 2 and 1 with a branch each, first all loads and then all sums (a branch per row
// costs more than it saves).  The rows keep their order.
static_assert(NT_MCHUNK <= 16, "the last chunk is walked in runs of 8, 4, 2 and 1 rows");
template <class GT, bool TABLE, int RUN>
__device__ inline void load_last(bool part, const StepParams& p, int j0, int nb, const Reach& at, typename GT::raw_t* raw) {
  if (nb & RUN) load_rows<GT, TABLE, RUN>(part, p, j0 + (nb & ~(2 * RUN - 1)), at, raw);
  if constexpr (RUN > 1) load_last<GT, TABLE, RUN / 2>(part, p, j0, nb, at, raw + RUN);
}
template <class GT, bool MOVES, int RUN>
__device__ inline void accumulate_last(int nb, typename GT::raw_t* raw, const Reach& at, const float* K, double* sb, float* q) {
  if (nb & RUN) chunk_accumulate<GT, MOVES, RUN>(raw, at, K, sb, q);
  if constexpr (RUN > 1) accumulate_last<GT, MOVES, RUN / 2>(nb, raw + RUN, at, K, sb, q);
}
template <class GT, bool MOVES, int RUN>
__device__ inline void moments_last(int nb, typename GT::raw_t* raw, const Reach& at, double* s, double* q) {
  if (nb & RUN) chunk_moments<GT, MOVES, RUN>(raw, at, s, q);
  if constexpr (RUN > 1) moments_last<GT, MOVES, RUN / 2>(nb, raw + RUN, at, s, q);
}

// How the walk of more than 32 bf16 rows in the class for long vectors keeps the blocks of a generation in step.  A chunk's first sum
// waits until its loads have arrived: without it, each sum starting as its row arrives, 64 / 128 / 512 rows at d = 2^24 took 414 / 734 /
// 2622 us, with it 401 / 716 / 2571; in short vectors it costs 1 to 5 %, with up to 32 rows 0.5 %, and below 48 rows all but four loads
// are the better count (40 rows with the mean 231 us, waiting for all of them 236).  And where a launch is a whole generation, so that
// every CU has four blocks, a wave of 48 rows or more pauses after each chunk: the memory system serves fewer requests at a time
// faster.  Without the pause / with 18 / with 30 times 64 cycles, us: fused step of 128 rows at 2^24 722 / 707 / 707, of 256 1339 / 1314 / 1316, of
// 512 2573 / 2522 / 2524, of 64 407 / 405 / 412 and at 1e8 2304 / 2288 / 2347, of 96 565 / 566 / 570; AdamW only of 256 rows at 2^23 690 / 661 / 656,
// of 48 175.0 / 173.3 / 172.8; 40 rows without and with it 289 and 291.  12 against 18: 128 rows at 2^24 710 / 706, 512 at 2^23 1293 / 1283, AdamW
// only of 256 663 / 660, 64 rows equal.  In a launch with fewer blocks the pause costs 3 %.
__device__ inline void chunk_wait(int J) {
  __builtin_amdgcn_sched_barrier(0);
  if (J >= NT_PAUSE_ROWS)
    __builtin_amdgcn_s_waitcnt(0x0f70);
  else if (J > 32)
    __builtin_amdgcn_s_waitcnt(0x0f70 | 4);   // vmcnt(4)
  __builtin_amdgcn_sched_barrier(0);
}
__device__ inline void chunk_pause(int J) {
  if (J < NT_PAUSE_ROWS || gridDim.x < NT_GENERATION / (NT_BLOCK_LARGE * NT_ITERS_LARGE * NT_VEC)) return;
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_sleep(18);
}

// bf16 rows of a matrix whose first row begins on 4 bytes and whose row stride is odd: every second row begins between two words, and
// loads of 8 bytes from there cost more than 12 from the word before, shifted.  What those read past the lane's coordinates, two bytes on
// either side, is in the matrix: the row is not the first, and the row goes on where the lanes end.  8 bytes -> 12, us: fused step of
// 20 / 64 / 128 / 512 rows at d = 300,001 8.6 / 16.5 / 25.8 / 81 -> 8.3 / 14.3 / 21.9 / 67, at 1,000,003 15.3 / 31.9 / 54.3 / 190 -> 14.4 / 28.8 /
// 50.4 / 179, statistics of 64 rows at 3e6 71.2 -> 68.8.  Where state or the mean is written, 8 bytes stay the better loads in long vectors: from
// 48 rows on, 64 / 128 at 1.8e6 56.7 / 101.6 -> 55.2 / 99.6, at 2e6 58.7 / 105.7 -> 58.6 / 107.5; 20 / 40 rows at 4e6 49.3 / 81.2 -> 48.6 / 80.0, 48
// rows 92.8 -> 93.8, 20 rows at 1e7 117 -> 119; and in the class for long vectors (64 rows at 1e7 304 -> 315, AdamW only, 128 rows 548 -> 575).
#define NT_ODD_ROWS 48
#define NT_ODD_COORDS (7ll << 18)
#define NT_ODD_COORDS_FEW (1ll << 22)    // below NT_ODD_ROWS rows
template <bool WRITES>
__device__ inline bool odd_rows(const StepParams& p, int64_t end) {
  if (WRITES && p.d >= (p.J >= NT_ODD_ROWS ? NT_ODD_COORDS : NT_ODD_COORDS_FEW)) return false;
  return (p.ld & 1) != 0 && ((uintptr_t)p.grads & 3) == 0 && end < p.d;
}
template <int N>
__device__ inline void load_odd(const StepParams& p, int j0, const Reach& r, BF16::raw_t* raw) {
  static_assert(N % 2 == 0, "pairs of rows");
  const uint32_t lane = r.u * BF16::ESIZE;
  RowWalk<BF16, false> row(p, j0, r.s0);
  u32x3 o[N / 2];
#pragma unroll
  for (int j = 0; j < N; j += 2) {
    raw[j] = BF16::ldraw(row.next() + lane);
    o[j / 2] = ld_nt<u32x3_words>(row.next() - 2 + lane);
  }
#pragma unroll
  for (int j = 1; j < N; j += 2) {
    const u32x3 x = o[j / 2];
    raw[j] = BF16::raw_t{__builtin_amdgcn_alignbit(x[1], x[0], 16), __builtin_amdgcn_alignbit(x[2], x[1], 16)};
  }
}

// All rows of the lane's coordinates: row sum, centred sum and sum of squares.  bf16 rows, by their moments (see centred).
template <class GT, bool TABLE, bool MOVES, bool WAITS, bool ODD = false>
__device__ inline void walk_moments(bool part, const StepParams& p, const Reach& at, double* S, float* M2, float* a) {
  constexpr int VEC = GT::VEC;
  const int J = p.J, segment = segment_rows(J);
  double Q[VEC], s[VEC], q[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) S[e] = Q[e] = s[e] = q[e] = 0.0;
  typename GT::raw_t raw[NT_MCHUNK];
  int j0 = 0, end = segment;
#pragma unroll 1
  for (; j0 + NT_MCHUNK <= J; j0 += NT_MCHUNK) {
    if (j0 == end) {
      end += segment;
      segment_end<VEC>(S, Q, s, q);
    }
    if constexpr (ODD)
      load_odd<NT_MCHUNK>(p, j0, at, raw);
    else
      load_rows<GT, TABLE, NT_MCHUNK>(part, p, j0, at, raw);
    if (WAITS) chunk_wait(J);
    chunk_moments<GT, MOVES, NT_MCHUNK>(raw, at, s, q);
    if (WAITS) chunk_pause(J);
  }
  if (j0 < J) {
    if (j0 == end) segment_end<VEC>(S, Q, s, q);
    load_last<GT, TABLE, 8>(part, p, j0, J - j0, at, raw);
    moments_last<GT, MOVES, 8>(J - j0, raw, at, s, q);
  }
  segment_end<VEC>(S, Q, s, q);
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    a[e] = (float)Q[e];
    M2[e] = centred(J, p.inv_J, S[e], Q[e]);
  }
}
// fp32 rows, whose squares need twice fp64's digits: every chunk shifted by the mean of the rows before it (see chunk_merge).
template <class GT, bool TABLE, bool MOVES>
__device__ inline void walk_shifted(bool part, const StepParams& p, const Reach& at, double* S, float* M2, float* a) {
  constexpr int VEC = GT::VEC;
  const int J = p.J;
  double sb[VEC];
  float K[VEC], q[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) a[e] = 0.f;
  typename GT::raw_t raw[NT_MCHUNK];
  // first chunk (J > NT_JCHUNK >= NT_MCHUNK - 1 here, so it is full), shifted by the first row
  load_rows<GT, TABLE, NT_MCHUNK>(part, p, 0, at, raw);
  if constexpr (MOVES) raw[0] = GT::moved(raw[0], at.sh);
#pragma unroll
  for (int e = 0; e < VEC; ++e) K[e] = GT::val(raw[0], e);
  chunk_clear<VEC>(sb, q);
  chunk_accumulate<GT, false, 1>(raw, at, K, sb, q);
  chunk_accumulate<GT, MOVES, NT_MCHUNK - 1>(raw + 1, at, K, sb, q);
#pragma unroll
  for (int e = 0; e < VEC; ++e) K[e] = chunk_merge(true, 0, NT_MCHUNK, 0.0, 1.0 / NT_MCHUNK, K[e], sb[e], q[e], S[e], M2[e], a[e]);
  double inv_j0 = 1.0 / NT_MCHUNK;
  int j0 = NT_MCHUNK;
#pragma unroll 1
  for (; j0 + NT_MCHUNK <= J; j0 += NT_MCHUNK) {
    load_rows<GT, TABLE, NT_MCHUNK>(part, p, j0, at, raw);
    chunk_clear<VEC>(sb, q);
    chunk_accumulate<GT, MOVES, NT_MCHUNK>(raw, at, K, sb, q);
    const double inv_n = 1.0 / (double)(j0 + NT_MCHUNK);
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      K[e] = chunk_merge(false, j0, NT_MCHUNK, inv_j0, inv_n, K[e], sb[e], q[e], S[e], M2[e], a[e]);
    inv_j0 = inv_n;
  }
  if (j0 < J) {
    const int nb = J - j0;
    load_last<GT, TABLE, 8>(part, p, j0, nb, at, raw);
    chunk_clear<VEC>(sb, q);
    accumulate_last<GT, MOVES, 8>(nb, raw, at, K, sb, q);
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      K[e] = chunk_merge(false, j0, nb, inv_j0, 0.0, K[e], sb[e], q[e], S[e], M2[e], a[e]);   // the last: K is not used again
  }
}

// The state update (and the gbar store) of a tile is deferred (see deferred_update): with many rows the writes are
// a few per cent of the traffic.
template <class GT, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool PART, bool END>
__device__ inline TileEnd tile_multi(bool part, const StepParams& p, int64_t tile, double (*red)[NT_NV], f32x4* gbs,
                                     uint32_t* ticket) {
  constexpr int VEC = GT::VEC;
  static_assert(VEC == 4, "one 16-byte LDS slot per lane and sweep");
  constexpr int TILE = BLOCK * VEC * ITERS;
  constexpr bool WRITES = (MODE != MODE_STATS) || GBAR;
  constexpr bool MOVES = PART && moves_rows<GT, 0, MODE, BLOCK, ITERS, TABLE, false>();
  constexpr bool ODDS = GT::ESIZE == 2 && !TABLE && !PART && (!WRITES || BLOCK * ITERS != NT_BLOCK_LARGE * NT_ITERS_LARGE);
  constexpr bool WAITS = WRITES && GT::ESIZE == 2 && BLOCK * ITERS == NT_BLOCK_LARGE * NT_ITERS_LARGE;
  LaneAcc acc;
#pragma unroll 1
  for (int it = 0; it < ITERS; ++it) {
    const Place pl = {tile * TILE + (int64_t)it * BLOCK * VEC, threadIdx.x * VEC};
    // a sweep or a wave that lies wholly past d adds nothing, and has no means to leave for the update
    if (PART && part && pl.s0 + (int64_t)__builtin_amdgcn_readfirstlane(threadIdx.x) * VEC >= p.d) break;
    double S[VEC];
    float M2[VEC], a[VEC];
    const Reach at = reach(PART && part, p, pl);
    if constexpr (ODDS) {
      if (odd_rows<WRITES>(p, pl.s0 + BLOCK * VEC))
        walk_moments<GT, TABLE, MOVES, WAITS, true>(PART && part, p, at, S, M2, a);
      else
        walk_moments<GT, TABLE, MOVES, WAITS>(PART && part, p, at, S, M2, a);
    } else if constexpr (GT::ESIZE == 2)
      walk_moments<GT, TABLE, MOVES, WAITS>(PART && part, p, at, S, M2, a);
    else
      walk_shifted<GT, TABLE, MOVES>(PART && part, p, at, S, M2, a);
    float gb[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) gb[e] = (float)(S[e] * p.inv_J);

    if constexpr (MODE != MODE_ADAMW) {
      float b[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float sf = (float)S[e];
        b[e] = sf * sf;
        coord_test(p.coord_thr, M2[e], gb[e], acc);
      }
      acc.A += (double)lane_tree<VEC>(a);
      acc.B += (double)lane_tree<VEC>(b);
      acc.C += (double)lane_tree<VEC>(M2);
    }
    if constexpr (WRITES) gbs[it * BLOCK + threadIdx.x] = f32x4{gb[0], gb[1], gb[2], gb[3]};
  }
  if constexpr (WRITES)
    return deferred_update<MODE, BLOCK, ITERS, GBAR, PART, END, MOVES>(p, tile, red, acc, gbs, ticket);
  else
    return tile_reduce<BLOCK, END>(acc, red, p.partials, tile, ticket);
}

// ---------------------------------------------------------------------------------------------
// Tile, more than 16 bf16 rows, in the shortest vectors (see NT_SPLIT_TILE): a block's waves share the rows too.  SPLIT waves walk one
// segment of the rows each at the same 256 coordinates; their sums meet in LDS, where each thread adds up the segments of its
// coordinate (or two coordinates, with two segments) in their order, with the bits of tile_multi.  Bound by what one CU reads, 45 GB/s:
// a tile of 512 rows takes 32 us, a MB at 33 GB/s; with a chunk split in halves, one in flight while the other is added up, 2 % more.
// ---------------------------------------------------------------------------------------------
template <int SPLIT, bool STATS>
struct SplitShared {
  double s[SPLIT][NT_SPLIT_TILE];
  double q[STATS ? SPLIT : 1][STATS ? NT_SPLIT_TILE : 1];
};
// x of the lane whose number differs in the last two bits as CTRL says (quad permutation)
template <int CTRL>
__device__ inline float quad(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
// lane_tree of the values of four neighbouring lanes
__device__ inline float quad_tree(float x) {
  x += quad<0xb1>(x);          // lanes 1 0 3 2
  return x + quad<0x4e>(x);    // lanes 2 3 0 1
}

template <class GT, int SPLIT, int MODE, bool TABLE, bool GBAR, bool END>
__device__ inline TileEnd tile_split(bool part, const StepParams& p, int64_t tile, double (*red)[NT_NV],
                                     SplitShared<SPLIT, MODE != MODE_ADAMW>& sh, uint32_t* ticket) {
  constexpr int VEC = GT::VEC, T = NT_SPLIT_TILE, BLOCK = SPLIT * T / VEC;
  constexpr int X = T / BLOCK;   // coordinates per thread
  static_assert(X * BLOCK == T, "whole tiles");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int mine = wave / (T / 256), col = wave % (T / 256);
  const int J = p.J, segment = segment_rows(J);
  const Place pl = {tile * T + col * 256, (uint32_t)lane * VEC};
  // a wave that lies wholly past d loads the vector's first group and moves all of it out
  const Reach at = pl.s0 < p.d ? reach(part, p, pl) : Reach{0, 0, 4};
  int j0 = mine * segment;
  const int end = j0 + segment < J ? j0 + segment : J;
  typename GT::raw_t raw[NT_MCHUNK];
  double s[VEC], q[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) s[e] = q[e] = 0.0;
  // the state of the coordinates that this thread finishes, on its way meanwhile
  bool own[X];
  float w[X], m[X], v[X];
#pragma unroll
  for (int x = 0; x < X; ++x) {
    const int i = threadIdx.x + x * BLOCK;
    own[x] = !part || tile * T + i < p.d;
    if constexpr (MODE != MODE_STATS) {
      w[x] = m[x] = v[x] = 0.f;
      if (own[x]) {
        w[x] = ld_nt<float>(scalar(p.w + tile * T) + i);
        m[x] = ld_nt<float>(scalar(p.m + tile * T) + i);
        v[x] = ld_nt<float>(scalar(p.v + tile * T) + i);
      }
    }
  }
  // 64 / 128 / 512 rows of odd stride, fused, 8 -> 12 bytes: at d = 20,001 9.9 / 13.7 / 37.8 -> 9.6 / 12.7 / 31.6 us, at 2e5 12.0 / 17.4 / 47.4 ->
  // 11.3 / 15.7 / 44.1; with two waves, and with AdamW only, the second loop costs even strides up to 6 and 4 %
  const bool odd = SPLIT == 4 && MODE != MODE_ADAMW && !TABLE && odd_rows<true>(p, pl.s0 + 256);
#pragma unroll 1
  for (; j0 + NT_MCHUNK <= end; j0 += NT_MCHUNK) {
    if (odd) {
      load_odd<NT_MCHUNK>(p, j0, at, raw);
      chunk_moments<GT, false, NT_MCHUNK>(raw, at, s, q);
      continue;
    }
    load_rows<GT, TABLE, NT_MCHUNK>(part, p, j0, at, raw);
    settle<GT, NT_MCHUNK, true>(part, pl, at, raw);
    chunk_moments<GT, false, NT_MCHUNK>(raw, at, s, q);
  }
  if (j0 < end) {
    load_last<GT, TABLE, 8>(part, p, j0, end - j0, at, raw);
    moments_last<GT, true, 8>(end - j0, raw, at, s, q);
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    sh.s[mine][col * 256 + lane * VEC + e] = s[e];
    if constexpr (MODE != MODE_ADAMW) sh.q[mine][col * 256 + lane * VEC + e] = q[e];
  }
  __syncthreads();
  LaneAcc acc;
  float gb[X];
#pragma unroll
  for (int x = 0; x < X; ++x) {
    const int i = threadIdx.x + x * BLOCK;
    double S = 0.0, Q = 0.0;
#pragma unroll
    for (int k = 0; k < SPLIT; ++k)
      if (k * segment < J) {
        S += sh.s[k][i];
        if constexpr (MODE != MODE_ADAMW) Q += sh.q[k][i];
      }
    gb[x] = (float)(S * p.inv_J);
    if constexpr (MODE != MODE_ADAMW) {
      const float sf = (float)S, c = centred(J, p.inv_J, S, Q);
      coord_test(p.coord_thr, c, gb[x], acc);
      const float ta = quad_tree((float)Q), tb = quad_tree(sf * sf), tc = quad_tree(c);
      if ((lane & 3) == 0) {
        acc.A += (double)ta;
        acc.B += (double)tb;
        acc.C += (double)tc;
      }
    }
  }
  TileEnd te = {0.0, 0};
  if constexpr (MODE != MODE_ADAMW) te = tile_reduce<BLOCK, END>(acc, red, p.partials, tile, ticket);
#pragma unroll
  for (int x = 0; x < X; ++x)
    if (own[x]) {
      const int i = threadIdx.x + x * BLOCK;
      if constexpr (MODE != MODE_STATS) {
        adamw_coord(p, gb[x], w[x], m[x], v[x]);
        __builtin_nontemporal_store(w[x], scalar(p.w + tile * T) + i);
        __builtin_nontemporal_store(m[x], scalar(p.m + tile * T) + i);
        __builtin_nontemporal_store(v[x], scalar(p.v + tile * T) + i);
      }
      if (GBAR && p.gbar) __builtin_nontemporal_store(gb[x], scalar(p.gbar + tile * T) + i);
    }
  return te;
}

// ---------------------------------------------------------------------------------------------
// Kernels.  A launch covers gridDim.x of the ntiles tile slots, from slot0 on, a block each; tiles below nfull are whole, and
// when the vector ends in a part of a tile (nfull = ntiles - 1), that one has slot 0, so that it overlaps with everything else.
// J_T = 0 selects the J > 16 row-walking variant, NT_SPLIT + n the one whose rows are shared by n waves.  (Walking tiles in a loop instead cost registers that every tile held: fused
// step of 8 bf16 rows 79 vector and 91 scalar registers, 76 and 50 without; AdamW only 86 scalar ones, 74 without.)
// ---------------------------------------------------------------------------------------------
template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool DEFER_T, bool COORD, bool PART, bool END>
__device__ inline TileEnd run_tile(bool part, const StepParams& p, int64_t tile, double (*red)[NT_NV], f32x4* gbs,
                                   uint32_t* ticket) {
  if constexpr (J_T == 0) {
    return tile_multi<GT, MODE, BLOCK, ITERS, TABLE, GBAR, PART, END>(part, p, tile, red, gbs, ticket);
  } else if constexpr (DEFER_T) {
    static_assert(!END || MODE == MODE_ADAMW, "steps with sums that write their own result are not in this class");
    tile_defer<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, PART>(p, tile, red, gbs);
    return {0.0, 0};
  } else {
    return tile_rows<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, COORD, PART, END>(part, p, tile, red, ticket);
  }
}

// Whether whole tiles run a copy of the walk of their own: more than 16 rows.  In the copy for part tiles every row is moved to its
// place (settle), which costs a short walk (statistics of 17 / 64 fp32 rows at d = 1e6 16.8 / 43.5 us in it, 15.5 / 42.1 beside it), so
// they do, but for short steps over tables that write their own result: there the second copy would need scratch memory.  With AdamW
// only nothing is moved, and the second copy is still the better one (64 bf16 rows 58.7 and 64.4 us at 2^21; 20 rows in tables 10.7
// and 11.6 at 1e6; 64 fp32 rows 510 and 527 at 1.2e7), but where one_copy says otherwise.
template <int MODE, int BLOCK, int ITERS, bool TABLE, bool END>
constexpr bool whole_copy() {
  return MODE == MODE_ADAMW || !TABLE || !END || BLOCK * ITERS == NT_BLOCK_LARGE * NT_ITERS_LARGE;
}

// GBAR = false compiles the gbar store out (statistics-only launch class, so that sweeps can overlap).
// DEFER_T: up to 16 rows with the state update deferred to the end of the tile (always so beyond 16 rows).
// COORD = false compiles the coordinate-wise test out (see plain_stats).
template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool DEFER_T, bool COORD, bool END>
__device__ inline TileEnd block_tile(const StepParams& p, int64_t nfull, int64_t ntiles, int64_t slot0, uint32_t* ticket) {
  constexpr int SPLIT = J_T > NT_SPLIT ? J_T - NT_SPLIT : 0;
  constexpr int TILE = SPLIT ? NT_SPLIT_TILE : BLOCK * GT::VEC * ITERS;
  static_assert(NT_TILE_MAX % TILE == 0, "tile sizes must divide NT_TILE_MAX");
  __shared__ double red[BLOCK / 64][NT_NV];
  // the means of a tile's sweeps wait here for the deferred state update (see deferred_update)
  constexpr bool DEFER = (J_T == 0 || DEFER_T) && ((MODE != MODE_STATS) || GBAR);
  static_assert(!DEFER_T || DEFER, "a deferred update needs something to write");
  __shared__ f32x4 gbs[DEFER ? ITERS * BLOCK + NT_LDS_PAD_LARGE / 16 : 1];
  const int64_t npart = ntiles - nfull;  // 0 or 1
  const int64_t t = slot0 + blockIdx.x;
  // rotate: the part tile (if any) first, then the whole tiles 0..nfull-1
  const bool part = t < npart;
  const int64_t tile = part ? nfull : t - npart;
  if constexpr (SPLIT > 0) {
    __shared__ SplitShared<SPLIT, MODE != MODE_ADAMW> sh;
    return tile_split<GT, SPLIT, MODE, TABLE, GBAR, END>(part, p, tile, red, sh, ticket);
  } else {
    constexpr bool ONE_COPY = one_copy<GT, J_T, MODE, BLOCK, ITERS, DEFER_T>();
    if (!ONE_COPY && !part && (J_T > 0 || whole_copy<MODE, BLOCK, ITERS, TABLE, END>()))
      return run_tile<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T, COORD, false, END>(false, p, tile, red, gbs, ticket);
    return run_tile<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T, COORD, true, END>(!ONE_COPY || part, p, tile, red, gbs, ticket);
  }
}

template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool DEFER_T = false, bool COORD = true>
__global__ __launch_bounds__(BLOCK) void k_step(StepParams p, int64_t nfull, int64_t ntiles, int64_t slot0) {
  block_tile<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T, COORD, false>(p, nfull, ntiles, slot0, nullptr);
}

// Blocks of 256 threads with one sweep, which fp32 rows take in the shortest vectors, are held to the 128 vector registers that four
// waves of a SIMD may have: with two more the compiler orders the walk worse (512 rows 1.13 times the time at d = 1000, 1.14 at 20,001).
// Not so read-only statistics over tables, which would need scratch memory.
template <int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR>
constexpr int waves_per_simd() {
  return BLOCK == 256 && ITERS == 1 && !(TABLE && MODE == MODE_STATS && !GBAR) ? 4 : 1;
}
// A step that writes its result itself: AdamW only, which has no sums; a single tile, whose partial is the total; or a few
// tiles, a block each, of which the last to finish adds up the partials in k_finalize's order.  A second kernel costs such a
// call 3.7 us on the host and some 2 on the GPU.  It is a kernel of its own because this tail in every kernel slows the long
// steps by 0.3 to 1 %.  What makes the handshake between blocks cheap is that it neither releases nor waits: see tile_reduce.
// (With marks beside the partials, which each block looks at after an agent-wide acquire of its own, the step of 256 tiles took
// 17.6 us against 13.2 for two launches at the time.)
template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool DEFER_T = false>
__global__ __launch_bounds__(BLOCK, (waves_per_simd<MODE, BLOCK, ITERS, TABLE, GBAR>())) void k_step_end(StepParams p, int64_t nfull, int64_t ntiles, int64_t slot0,
                                                    Finish fin) {
  const TileEnd end = block_tile<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T, true, true>(p, nfull, ntiles, slot0,
                                                                                                      leaf_of(fin.ticket, ntiles));
  Totals tot;
  totals_clear(tot);
  if constexpr (MODE == MODE_ADAMW) {
    if (slot0 != 0 || blockIdx.x != 0) return;
  } else if (!fin.ticket) {
    // the only tile's partial, added to zero as in k_finalize: the addition leaves finite sums as they are and turns an
    // infinite one into NaN, so sums that overflow (and the clipping factor, which is 1 then) read the same whatever the
    // number of tiles
    const dd t = dd_add(dd{0.0, 0.0}, dd{end.value, 0.0});
    tot.s[0] = t;
    tot.s[1] = ahead<1>(t);
    tot.s[2] = ahead<2>(t);
    tot.s[3] = ahead<3>(t);
    tot.mx = ahead<4>(end.value);
  } else {
    // The last block to count itself finds every partial in memory; it has invalidated its caches, which may hold older ones.
    __shared__ bool last;
    __shared__ double sh[NT_FIN_THREADS / 64][2 * NT_NV];
    if (threadIdx.x == 0) last = last_block(fin.ticket, (uint32_t)ntiles, end.before);
    __syncthreads();
    if (!last) return;
    block_totals<NT_FIN_THREADS, false>(p.partials, ntiles, sh, tot);
  }
  if (threadIdx.x == 0) write_record(tot, fin.q, fin.out, fin.hdr, fin.hdr_out);
}

// ---------------------------------------------------------------------------------------------
// Reduction of the tile partials.
// ---------------------------------------------------------------------------------------------
// Long vectors: block g adds the partials of the g-th group of tiles into one double-double record, and the last block to finish adds
// up the records and takes the decision.  Records are handed over like the partials of k_step_end (tile_reduce), at a counter
// in the workspace that the step's own kernel has set to zero: a graph takes it along.  (With a device-wide release by every
// block, which writes back all of an XCD's L2, one launch took 26 us at 15 groups; as two launches 4.6 + 4.5.)
__global__ __launch_bounds__(NT_FIN_THREADS) void k_reduce_end(const double* tiles, int64_t ntiles, double* groups, DecideParams q,
                                                               nt_result* out, WsRecord hdr, WsRecord* hdr_out) {
  __shared__ double sh[NT_FIN_THREADS / 64][2 * NT_NV];
  __shared__ bool last;
  const int64_t per = group_tiles(ntiles), t0 = (int64_t)blockIdx.x * per;
  Totals tot;
  totals_clear(tot);
  block_totals<NT_FIN_THREADS, false>(tiles + NT_NV * t0, ntiles - t0 < per ? ntiles - t0 : per, sh, tot);
  if (threadIdx.x == 0) {
    double* rec = groups + 2 * NT_NV * (int64_t)blockIdx.x;
    auto hand_on = [](double* to, double x) { __hip_atomic_store(to, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
#pragma unroll
    for (int k = 0; k < NT_NSUM; ++k) {
      hand_on(rec + 2 * k, tot.s[k].hi);
      hand_on(rec + 2 * k + 1, tot.s[k].lo);
    }
    hand_on(rec + 2 * NT_NSUM, tot.mx);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    last = count_up((uint32_t*)(tiles - NT_WS_HEADER + NT_WS_COUNTER)) == gridDim.x - 1;
    if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
  if (!last) return;
  totals_clear(tot);
  block_totals<NT_FIN_THREADS, true>(groups, gridDim.x, sh, tot);
  if (threadIdx.x == 0) write_record(tot, q, out, hdr, hdr_out);
}

// One block: tile partials -> A, B, C in double-double, then the decision.
__global__ __launch_bounds__(NT_FIN_THREADS) void k_finalize(const double* in, int64_t n, DecideParams q, nt_result* out,
                                                             WsRecord hdr, WsRecord* hdr_out) {
  __shared__ double sh[NT_FIN_THREADS / 64][2 * NT_NV];
  const bool stats = (q.flags & NT_DO_STATS) != 0;
  Totals tot;
  totals_clear(tot);
  if (stats) block_totals<NT_FIN_THREADS, false>(in, n, sh, tot);
  if (threadIdx.x != 0) return;
  write_record(tot, q, out, hdr, hdr_out);
}

// Threads of the per-layer kernel: 1024, but where more than 16 fp32 rows are walked, for which 128 vector registers are too few.
template <class GT, bool MANY>
constexpr int layer_threads() {
  return MANY && GT::ESIZE == 4 ? 512 : 1024;
}
// What a coordinate adds to the sums of its piece.
__device__ inline void piece_add(const StepParams& p, double S, float M2, float a, LaneAcc& acc) {
  const float gb = (float)(S * p.inv_J), sf = (float)S;
  acc.A += (double)a;
  acc.B += (double)(sf * sf);
  acc.C += (double)M2;
  coord_test(p.coord_thr, M2, gb, acc);
}
// Sums over the coordinates [plo, phi), up to 16 rows: one coordinate per thread.
template <class GT, bool TABLE, int J_T>
__device__ inline void piece_sums(const StepParams& p, int64_t plo, int64_t phi, LaneAcc& acc) {
#pragma unroll 2
  for (int64_t i = plo + threadIdx.x; i < phi; i += layer_threads<GT, false>()) {
    double S;
    float M2, a;
    coord_stats<GT, TABLE, J_T>(p, i, S, M2, a);
    piece_add(p, S, M2, a, acc);
  }
}
// Sums over the coordinates of two pieces [lo, hi), more than 16 rows, by the tiles' own walks: a wave takes 256 coordinates, the first
// piece's before the second's.  With a coordinate per thread, whose rows are loaded two or four bytes at a time, and one piece after the other,
// the table of 148 layers, 128 bf16 rows, d = 1,000,003 took 172 us, so 39; 12 layers, 512 rows, 100,003 556 and 56; 300 layers, 64
// fp32 rows, 300,007 108 and 29.  (Up to 16 rows this way is 0.9 to 1.2 times as fast as a coordinate per thread.)
template <class GT, bool TABLE>
__device__ inline void pieces_walk(const StepParams& p, const int64_t (&lo)[2], const int64_t (&hi)[2], LaneAcc& acc) {
  constexpr int SPAN = 64 * NT_VEC;
  int64_t from[2], spans[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    from[k] = lo[k] & ~(int64_t)(NT_VEC - 1);
    spans[k] = lo[k] < hi[k] ? (hi[k] - from[k] + SPAN - 1) / SPAN : 0;
  }
#pragma unroll 1
  for (int64_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); w < spans[0] + spans[1]; w += layer_threads<GT, true>() / 64) {
    const bool second = w >= spans[0];
    const Place pl = {second ? from[1] + (w - spans[0]) * SPAN : from[0] + w * SPAN, (threadIdx.x & 63) * NT_VEC};
    const int64_t first = second ? lo[1] : lo[0], end = second ? hi[1] : hi[0];
    const Reach at = reach(true, p, pl);
    double S[NT_VEC];
    float M2[NT_VEC], a[NT_VEC];
    if constexpr (GT::ESIZE == 2)
      walk_moments<GT, TABLE, true, false>(true, p, at, S, M2, a);
    else
      walk_shifted<GT, TABLE, true>(true, p, at, S, M2, a);
#pragma unroll
    for (int e = 0; e < NT_VEC; ++e)
      if (pl.i0() + e >= first && pl.i0() + e < end) piece_add(p, S[e], M2[e], a[e], acc);
  }
}

// Per-layer statistics from what a step left behind.  Layer l owns coordinates offsets[l] .. offsets[l+1]-1.
// Block l adds the partials of the tiles that lie wholly inside the layer (through the group partials
// where a whole group does) and recomputes, from the gradient rows, the at most two pieces at the layer's
// ends that cover only part of a tile; then the layer's own statistic (Alg. 1's T on the layer's
// coordinates) is formed.  Offsets are clamped into [0, d], so every access stays in bounds whatever
// the table holds; a clamped or descending pair is reported in the layer's status.
template <class GT, bool TABLE, bool MANY>
__global__ __launch_bounds__((layer_threads<GT, MANY>())) void k_layer_stats(StepParams p, const int64_t* offsets, const double* ws,
                                                                           nt_layer_stats* out) {
  constexpr int THREADS = layer_threads<GT, MANY>();
  __shared__ double sh[THREADS / 64][2 * NT_NV];
  const WsHeader h = *(const WsHeader*)ws;
  const int l = blockIdx.x;
  const double nan = __builtin_nan("");
  const bool usable = h.magic == NT_WS_MAGIC && h.has_stats && h.d == p.d && h.J == (int64_t)p.J &&
                      h.gdtype == (GT::ESIZE == 4 ? (int32_t)NT_F32 : (int32_t)NT_BF16) && h.tile_coords > 0;
  int64_t lo = offsets[l], hi = offsets[l + 1];
  uint32_t status = 0;
  if (lo < 0 || lo > p.d || hi < lo || hi > p.d) status |= NT_STATUS_BAD_RANGE;
  lo = lo < 0 ? 0 : (lo > p.d ? p.d : lo);
  hi = hi < lo ? lo : (hi > p.d ? p.d : hi);
  if (!usable) {
    if (threadIdx.x == 0) {
      nt_layer_stats r;
      r.A = r.B = r.C = r.gbar_sq = r.var_l1 = r.T = nan;
      r.coord_max_ratio = -1.0;
      r.n = hi - lo;
      r.coord_fail = -1;
      r.pass = 1;
      r.status = status | NT_STATUS_NO_STATS;
      out[l] = r;
    }
    return;
  }
  p.coord_thr = (float)h.coord_thr;
  const int64_t tc = h.tile_coords;
  const int64_t first = (lo + tc - 1) / tc;                      // first tile that starts at or after lo
  const int64_t head_end = first * tc < hi ? first * tc : hi;    // head piece [lo, head_end)
  int64_t last = first, tail_lo = hi;                            // whole tiles [first, last), tail piece [tail_lo, hi)
  if (head_end < hi) {
    last = hi / tc;
    tail_lo = last * tc;
  }
  LaneAcc piece;
  const int64_t plo[2] = {lo, tail_lo}, phi[2] = {head_end, hi};
  if constexpr (MANY) {
    pieces_walk<GT, TABLE>(p, plo, phi, piece);
  } else {
    for (int part = 0; part < 2; ++part) {
      if (plo[part] >= phi[part]) continue;
#define NT_CASE(JJ) \
  case JJ:          \
    piece_sums<GT, TABLE, JJ>(p, plo[part], phi[part], piece); \
    break;
      switch (p.J) {
        NT_CASE(2) NT_CASE(3) NT_CASE(4) NT_CASE(5) NT_CASE(6) NT_CASE(7) NT_CASE(8) NT_CASE(9)
        NT_CASE(10) NT_CASE(11) NT_CASE(12) NT_CASE(13) NT_CASE(14) NT_CASE(15) NT_CASE(16)
      }
#undef NT_CASE
    }
  }
  Totals acc;
  acc.s[0] = {piece.A, 0.0};
  acc.s[1] = {piece.B, 0.0};
  acc.s[2] = {piece.C, 0.0};
  acc.s[3] = {(double)piece.nfail, 0.0};
  acc.mx = (double)piece.rmax;
  const double* tiles = ws + NT_WS_HEADER;
  const double* groups = tiles + NT_NV * h.ntiles;
  const int64_t per = group_tiles(h.ntiles), g0 = (first + per - 1) / per, g1 = last / per;
  if (h.ngroups == (h.ntiles + per - 1) / per && g0 < g1) {   // a workspace kept from a build with other groups is read tile by tile
    totals_accumulate<THREADS, false>(tiles + NT_NV * first, g0 * per - first, acc);
    totals_accumulate<THREADS, true>(groups + 2 * NT_NV * g0, g1 - g0, acc);
    totals_accumulate<THREADS, false>(tiles + NT_NV * g1 * per, last - g1 * per, acc);
  } else {
    totals_accumulate<THREADS, false>(tiles + NT_NV * first, last - first, acc);
  }
  Totals tot;
  block_totals_finish<THREADS>(acc, sh, tot);
  if (threadIdx.x != 0) return;
  nt_result t;
  t.A = tot.s[0].hi;
  t.B = tot.s[1].hi;
  t.C = tot.s[2].hi;
  t.status = 0;
  DecideParams q = h.q;
  q.b_max = 0;
  q.round_to = 1;
  q.max_norm = 0.0;
  decide(q, &t);
  nt_layer_stats r;
  r.A = t.A;
  r.B = t.B;
  r.C = t.C;
  r.gbar_sq = t.gbar_sq;
  r.var_l1 = t.var_l1;
  r.T = t.T;
  r.coord_max_ratio = (h.coord_thr >= 0.0) ? tot.mx : -1.0;
  r.n = hi - lo;
  r.coord_fail = (h.coord_thr >= 0.0) ? (int64_t)tot.s[3].hi : -1;
  r.pass = t.pass;
  r.status = status | (t.status & (NT_STATUS_NONFINITE | NT_STATUS_ZERO_GRAD_NORM | NT_STATUS_T_SATURATED));
  out[l] = r;
}

// Phase 2 of the clipped variant: AdamW on scale * gbar, gbar read from memory.  One sweep per block, 4 coordinates
// per lane.
template <bool PART>
__device__ inline void adamw_gbar_sweep(StepParams& p, const float* gbar, float scale, const Place& pl) {
  u32x4 sg, state[3];
  p.grads = gbar;   // as the only row
  const Reach at = reach(PART, p, pl);
  load_sweep<F32, false, 1, true>(PART, p, 0, at, &sg, state);
  float gb[NT_VEC];
#pragma unroll
  for (int e = 0; e < NT_VEC; ++e) gb[e] = scale * __builtin_bit_cast(float, (uint32_t)sg[e]);
  adamw_store(PART, p, at, gb, state);
}
__global__ __launch_bounds__(NT_AUX_BLOCK) void k_adamw_gbar(StepParams p, const float* gbar, float grad_scale,
                                                         const nt_result* res, int64_t block0) {
  float scale = grad_scale;
  if (res) scale *= (float)res->clip_coef;
  const Place pl = {(block0 + blockIdx.x) * NT_AUX_BLOCK * NT_VEC, threadIdx.x * NT_VEC};
  if (pl.s0 + NT_AUX_BLOCK * NT_VEC <= p.d)
    adamw_gbar_sweep<false>(p, gbar, scale, pl);
  else
    adamw_gbar_sweep<true>(p, gbar, scale, pl);
}

__global__ __launch_bounds__(NT_AUX_BLOCK) void k_copy16(f32x4* dst, const u32x4* src, int64_t n16) {
  for (int64_t i = (int64_t)blockIdx.x * NT_AUX_BLOCK + threadIdx.x; i < n16; i += (int64_t)gridDim.x * NT_AUX_BLOCK) {
    const u32x4 x = ld16(src + i);
    st16(dst + i, __builtin_bit_cast(f32x4, x));
  }
}


// ---------------------------------------------------------------------------------------------
// Yardstick: R8 row-like read streams (8 bytes per lane, like four bfloat16 values of a gradient row), R16 read
// streams and W written streams (16 bytes per lane, like four fp32 values of w, m or v; RMW: read first, as an
// in-place update does), all walked in step by one block per 4096 coordinates with the step kernel's load and
// store instructions and no arithmetic beyond an exclusive-or that keeps every load alive.  It shows what
// the memory system gives for a mix of streams, independent of the step's arithmetic.
// ---------------------------------------------------------------------------------------------
#define NT_CALIB_MAX_R8 16
#define NT_CALIB_MAX_R16 12
#define NT_CALIB_MAX_W 4
struct CalibStreams {
  const char* r8[NT_CALIB_MAX_R8];
  const char* r16[NT_CALIB_MAX_R16];
  char* w[NT_CALIB_MAX_W];
  uint32_t* sink;   // spare word behind the streams; read-only mixes store to it when a load hits one magic value
};

template <int R8, int R16, int W, bool RMW>
__global__ __launch_bounds__(NT_AUX_BLOCK) void k_calib_streams(CalibStreams s, int64_t group0, int64_t group1) {
  for (int64_t i = group0 + (int64_t)blockIdx.x * NT_AUX_BLOCK + threadIdx.x; i < group1; i += (int64_t)gridDim.x * NT_AUX_BLOCK) {
    u32x2 a[R8 > 0 ? R8 : 1];
    u32x4 b[R16 > 0 ? R16 : 1];
    u32x4 c[W > 0 ? W : 1];
#pragma unroll
    for (int k = 0; k < R8; ++k) a[k] = ld_nt<u32x2>(s.r8[k] + 8 * i);
#pragma unroll
    for (int k = 0; k < R16; ++k) b[k] = ld16(s.r16[k] + 16 * i);
    if constexpr (RMW) {
#pragma unroll
      for (int k = 0; k < W; ++k) c[k] = ld16(s.w[k] + 16 * i);
    }
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < R8; ++k) acc ^= a[k][0] ^ a[k][1];
#pragma unroll
    for (int k = 0; k < R16; ++k) acc ^= b[k][0] ^ b[k][1] ^ b[k][2] ^ b[k][3];
#pragma unroll
    for (int k = 0; k < W; ++k) {
      u32x4 o = {acc, acc + 1u, acc + 2u, acc + 3u};
      if constexpr (RMW) o ^= c[k];
      st16(s.w[k] + 16 * i, __builtin_bit_cast(f32x4, o));
    }
    if constexpr (W == 0) {
      if (acc == 0x9e3779b9u) *s.sink = acc;   // data-dependent, so the loads cannot be dropped
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
inline int hip_code(hipError_t e) { return e == hipSuccess ? NT_OK : NT_ERR_HIP_BASE - (int)e; }

int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    __atomic_store_n(&cached[dev], n, __ATOMIC_RELAXED);
  }
  return n;
}

// Launch class of a call: block size and sweeps per tile.  Every tile is block * NT_VEC * sweeps
// coordinates and divides NT_TILE_MAX.
struct TileCfg {
  int block, iters;
  int64_t coords() const { return (int64_t)block * NT_VEC * iters; }
};
// Kernels without the coordinate-wise test, for calls that do not ask for it: its branch per coordinate keeps a sweep's
// instructions from being scheduled together and consecutive sweeps from overlapping, which shows where there is little
// traffic per coordinate.  Measured without against with it, GB/s at d = 2e8..3e8: read-only statistics of 2 / 4 / 8 bf16
// rows 6250 / 6810 / 6990 against 3940 / 6040 / 6960; statistics with gbar, 2 / 3 / 4 rows 5900 / 6040 / 6130 against
// 5350 / 5730 / 5290, 5 and 6 rows -5 and -1 %; fused step, 2 / 3 / 4 bf16 and 2 fp32 rows 5920 / 5870 / 5940 / 5800
// against 5550 / 5560 / 5790 / 5600, 5 to 8 bf16 rows -1 .. +0.8 %, 3 to 5 fp32 rows -3 .. -5 %.
constexpr bool plain_stats(int esize, int J, int mode, bool gbar) {
  return (mode == MODE_STATS && !gbar) || (mode != MODE_ADAMW && J * esize <= 8);
}
// ... and how far, in coordinates of the call, the same holds for statistics with more bytes of rows (short vectors without
// gbar among them, which run the kernels with it).  Without against with the test, us: 4 fp32 rows and gbar 24.1 / 26.8 at
// d = 5e6, 69.1 / 71.0 at 2^24, 344 / 334 at 1e8; 8 bf16 rows 22.5 / 23.1 at 2^22, 105.4 / 106.3 at 3e7, 628 / 625 at 2e8;
// 13 / 14 bf16 rows 12.3 / 12.8 and 12.6 / 13.0 at 2^20, 5 to 16 rows -0.3 .. -5 % up to 2^22, 14 rows +2 % at 5e6 .. 7e6.
constexpr int64_t plain_coords(int esize, int J, int mode) {
  return mode != MODE_STATS || J * esize < 16 ? 0 : J * esize == 16 ? 1ll << 25 : 1ll << 22;
}
constexpr int defer_row_bytes(int mode) { return mode == MODE_ADAMW ? NT_DEFER_ROW_BYTES_ADAMW : NT_DEFER_ROW_BYTES; }
// Which launch class a call takes beside its row count, dtype and mode: CLS_LONG, the classes for long vectors
// (large tiles, state update deferred, one generation of blocks per launch); CLS_SHORT, read-only statistics of up to
// 16 rows over a short vector, and anything of more rows over a shorter one; else CLS_BASE.  esize: bytes per gradient element; d_whole: length of the
// vector the call is a part of (its own d unless the caller said otherwise), so that the parts of a vector and the
// vector itself are cut into the same tiles.
enum { CLS_BASE = 0, CLS_LONG = 1, CLS_SHORT = 2, CLS_TINY = 3 };
// More than 16 rows: whether a vector of d coordinates is better walked in whole generations of blocks than in short tiles.  What
// is left over after the last full generation runs by itself on a few CUs, with two waves a block, and takes about as long whether it
// is little or much; short tiles take 5 to 10 % more per coordinate.  So what is left over decides: it has to be nothing or more than a
// part of a generation that shrinks with the number of full ones, and shrinks the sooner the more bytes a tile moves.  Generations
// against short tiles, us, fused step: 64 bf16 rows 158 / 173 at d = 6.3e6, 177 / 189 at 7e6, 291 / 226 at 8.4e6 (just past one),
// 298 / 274 at 1e7, 319 / 310 at 1.15e7, 326 / 348 at 1.3e7, 478 / 448 at 1.68e7 (just past two), 486 / 482 at 1.75e7, 504 / 517 at 1.9e7,
// 604 / 681 at 2.5e7; 40 rows 138 / 135 at 6.6e6; 256 rows 1021 / 744 at 8.4e6, 1116 / 1020 at 1.15e7, 1132 / 1142 at 1.3e7; 64 fp32 rows 306 /
// 317 at 6.3e6, 481 / 449 at 9e6, 477 / 518 at 1.04e7; 24 bf16 rows, whose generations are short-lived, 237 / 206 at 1.68e7, 251 / 236 at
// 1.9e7, 263 / 288 at 2.2e7.  Statistics with the mean, 128 bf16 rows 275 / 265 at 6.5e6, 64 fp32 rows 298 / 287; AdamW only, 64 fp32 rows
// 298 / 316 at 6.3e6, 449 / 469 at 9.5e6, 457 / 508 at 1.04e7, 128 bf16 rows 524 / 545 at 1.15e7, 64 rows 459 / 467 at 1.78e7.  Just past
// three generations and more, short tiles have not been measured.
// The generation is a constant, not the device's: the parts of a vector are cut into the same tiles wherever they run.
inline bool generations_pay(int64_t J, int esize, int mode, int64_t d) {
  constexpr int64_t G = NT_GENERATION;
  const int64_t full = d / G, left = d % G;
  const bool bf16 = esize == 2, adamw = mode == MODE_ADAMW;
  if (J <= 32) return full > 2 || (full == 2 && (J <= NT_FEW_ROWS || !bf16 || left == 0 || left > G / 4));
  if (full == 0) return left >= ((mode == MODE_FULL && J * esize >= 96) || (adamw && !bf16) ? G * 3 / 4 : G * 13 / 16);
  if (left == 0 || full > 2) return true;
  if (full == 1) return left > (bf16 ? (adamw && J >= 64 ? G * 5 / 16 : G * 3 / 8) : adamw ? G / 16 : mode == MODE_FULL ? G / 8 : G / 4);
  return !bf16 || left > (adamw && J >= 64 ? G / 16 : G / 8);
}
inline bool one_tile(int64_t J, int esize, int mode, int64_t d_whole) {
  if (mode == MODE_ADAMW || d_whole > NT_BLOCK_MANY_TINY * NT_ITERS_MANY_TINY * NT_VEC) return false;
  if (d_whole <= NT_SPLIT_TILE) return esize == 2 && J <= NT_ONE_TILE_ROWS_HALF;
  return J <= (esize == 2 ? NT_ONE_TILE_ROWS : NT_ONE_TILE_ROWS_32);
}
inline int launch_class(int64_t J, int esize, int mode, bool gbar, int64_t d_whole) {
  if (J > NT_JCHUNK && d_whole <= NT_SPLIT_COORDS) return one_tile(J, esize, mode, d_whole) ? CLS_SHORT : CLS_TINY;
  if (J > NT_JCHUNK && d_whole <= (J <= 32 && esize == 2 && mode != MODE_ADAMW ? NT_MANY_TINY_COORDS_32 : NT_MANY_TINY_COORDS)) return CLS_SHORT;
  if (mode == MODE_STATS && !gbar) return (J <= NT_JCHUNK && d_whole < NT_STATS_SHORT_COORDS) ? CLS_SHORT : CLS_BASE;
  if (J > NT_JCHUNK) return generations_pay(J, esize, mode, d_whole) ? CLS_LONG : CLS_BASE;
  return (J * esize >= defer_row_bytes(mode) && d_whole >= NT_DEFER_COORDS) ? CLS_LONG : CLS_BASE;
}
inline TileCfg tile_cfg(int64_t J, int esize, int mode, bool gbar, int64_t d_whole) {
  const int cls = launch_class(J, esize, mode, gbar, d_whole);
  if (J > NT_JCHUNK) {
    if (cls == CLS_TINY) return {NT_SPLIT_TILE / NT_VEC, 1};
    if (cls == CLS_SHORT) return {NT_BLOCK_MANY_TINY, NT_ITERS_MANY_TINY};
    if (mode == MODE_STATS && !gbar) return {NT_BLOCK_LARGE_STATS, NT_ITERS_LARGE_STATS};
    return cls == CLS_LONG ? TileCfg{NT_BLOCK_LARGE, NT_ITERS_LARGE} : TileCfg{NT_BLOCK_MANY_SHORT, NT_ITERS_MANY_SHORT};
  }
  if (cls == CLS_LONG) return {NT_BLOCK_DEFER, NT_ITERS_DEFER};
  if (mode == MODE_STATS && (gbar || cls == CLS_SHORT)) return {NT_BLOCK_STATS_GBAR, NT_ITERS_STATS_GBAR};
  if (mode == MODE_STATS) return {NT_BLOCK_STATS, NT_ITERS_STATS};
  if (mode == MODE_ADAMW) return {NT_BLOCK_ADAMW, NT_ITERS_ADAMW};
  return {NT_BLOCK, NT_ITERS};
}
static_assert(NT_BLOCK_FEW * NT_ITERS_FEW == NT_BLOCK_LARGE * NT_ITERS_LARGE, "both many-row shapes own the same tile");
static_assert(NT_BLOCK_DEFER * NT_ITERS_DEFER >= NT_BLOCK * NT_ITERS &&
                  NT_BLOCK_DEFER * NT_ITERS_DEFER >= NT_BLOCK_ADAMW * NT_ITERS_ADAMW &&
                  NT_BLOCK_DEFER * NT_ITERS_DEFER >= NT_BLOCK_STATS_GBAR * NT_ITERS_STATS_GBAR,
              "the deferred class never has more tiles than the class it replaces: the workspace is sized by the latter");
// tile slots per launch of the step kernel for the same classes (at least one, at most all)
inline int64_t launch_tiles(int64_t J, int esize, int mode, bool gbar, int cls, int64_t d, int64_t ntiles) {
  int64_t coords;
  if (J > NT_JCHUNK || cls != CLS_BASE)
    return ntiles;   // one launch, or generations of blocks: launch_step_shape knows the kernel's occupancy
  else if (mode == MODE_STATS)
    coords = gbar ? NT_CHUNK_STATS_GBAR : NT_CHUNK_STATS;
  else if (mode == MODE_ADAMW)
    coords = d < NT_LONG_COORDS ? NT_CHUNK_ADAMW : NT_CHUNK_ADAMW_LONG;
  else
    coords = J * esize <= 8 ? NT_CHUNK_FULL_FEW : NT_CHUNK_FULL;
  const int64_t n = coords / tile_cfg(J, esize, mode, gbar, 0).coords();
  return (n < 1 || n > ntiles) ? ntiles : n;
}
// dynamic LDS of a kernel with blocks of 1024 threads, which decides how many of them a CU holds (see NT_ONE_BLOCK_LDS)
inline unsigned one_block_lds(int64_t J, int esize, int mode, int64_t d) {
  const bool one = mode == MODE_ADAMW ? J * esize >= 16 && d > (1ll << 23) && d < NT_LONG_COORDS
                                      : J * esize >= (esize == 4 ? 12 : 16) && d > (esize == 4 ? 1ll << 24 : 1ll << 25);
  return one ? NT_ONE_BLOCK_LDS : 0;
}
// ... and of statistics that store the mean (see NT_TWO_BLOCK_LDS)
inline unsigned stats_gbar_lds(int64_t J, int esize, int64_t d) {
  if (d <= NT_HOLD_GBAR_COORDS || J * esize < 10) return 0;
  return J * esize < 12 ? NT_THREE_BLOCK_LDS : NT_TWO_BLOCK_LDS;
}
// smallest tile any mode and gradient type uses for this J, where the vector is longer than NT_SPLIT_COORDS if J > 16: sizes the workspace
inline int64_t min_tile_coords(int64_t J) {
  int64_t best = NT_TILE_MAX;
  const int modes[3] = {MODE_FULL, MODE_STATS, MODE_ADAMW};
  for (int m : modes)
    for (int g = 0; g < 2; ++g)
      for (int esize = 2; esize <= 4; esize += 2) {
        for (int64_t d_whole : {J > NT_JCHUNK ? NT_SPLIT_COORDS + 1 : 0, NT_DEFER_COORDS}) {   // shortest and longest
          const int64_t c = tile_cfg(J, esize, m, g != 0, d_whole).coords();
          if (c < best) best = c;
        }
      }
  return best;
}

bool hyper_ok(const nt_hyper* h, int64_t J) {
  if (!h) return false;
  const uint32_t known = NT_DO_STATS | NT_DO_ADAMW | NT_PARTIAL | NT_WRITE_GBAR | NT_COORD_TEST | NT_ONE_PASS;
  if (h->flags & ~known) return false;
  if (!(h->flags & (NT_DO_STATS | NT_DO_ADAMW))) return false;
  if ((h->flags & (NT_PARTIAL | NT_COORD_TEST)) && !(h->flags & NT_DO_STATS)) return false;
  if (!(h->eta > 0.0) || !std::isfinite(h->eta)) return false;
  if (h->b_k < 1 || h->b_max < 0 || h->round_to < 1 || h->round_to > NT_ROUND_TO_MAX) return false;
  if (h->ddof != 0 && h->ddof != 1) return false;
  if (J - h->ddof < 1) return false;
  if (h->flags & NT_DO_ADAMW) {
    if (h->step < 1) return false;
    if (!(h->lr >= 0.0) || !std::isfinite(h->lr)) return false;
    if (!(h->beta1 >= 0.0 && h->beta1 < 1.0) || !(h->beta2 >= 0.0 && h->beta2 < 1.0)) return false;
    if (!(h->eps >= 0.0) || !std::isfinite(h->eps)) return false;
    if (!(h->weight_decay >= 0.0) || !std::isfinite(h->weight_decay)) return false;
  }
  return true;
}

// How many blocks of a kernel with a deferred update a CU holds at a time (the runtime's occupancy query, asked
// once per device and kernel; 4 if it cannot be had).
template <auto KERNEL, int BS>
int blocks_per_cu() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 4;
  int n = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
  if (n <= 0) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, KERNEL, BS, 0) != hipSuccess || n < 1) {
      (void)hipGetLastError();
      n = 4;
    }
    __atomic_store_n(&cached[dev], n, __ATOMIC_RELAXED);
  }
  return n;
}

// The kernel of a launch class: with AdamW only the one that writes the result.
template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool DEFER_T = false>
constexpr auto step_kernel() {
  if constexpr (MODE == MODE_ADAMW)
    return k_step_end<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T>;
  else
    return k_step<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T>;
}
// FEW_TILES: a class that calls of one or a few tiles take; it has kernels that write the result (with the coordinate-wise
// test, whether it is asked for or not: up to 2^20 coordinates it costs nothing measurable).  Beyond 16 rows that is the class of the
// shortest vectors and, for short parts of longer ones, matrices in the classes of short tiles (2000 of 2^22 coordinates, fused step of
// 17 bf16 rows 7.5 us, 9.4 with a second launch; statistics of 33 rows, 700 of 2^30, 5.4 and 7.5).  Returns whether the launched
// kernel writes the result when it is the step's last: the caller's only source for that, so that no step can end without one.
template <class GT, int J_T, int MODE, int BLOCK, int ITERS, bool TABLE, bool GBAR, bool FEW_TILES, bool DEFER_T = false,
          bool COORD = true>
bool launch_tiles_of(const StepParams& p, int64_t nfull, int64_t ntiles, int64_t slot0, unsigned grid, const Finish& fin,
                     hipStream_t st) {
  unsigned lds = 0;
  if (BLOCK == 1024) lds = one_block_lds(p.J, GT::ESIZE, MODE, p.d);
  if (MODE == MODE_STATS && GBAR && J_T > 0 && !DEFER_T) lds = stats_gbar_lds(p.J, GT::ESIZE, p.d);
  if constexpr (MODE == MODE_ADAMW || FEW_TILES) {
    if (fin.out) {
      hipLaunchKernelGGL((k_step_end<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T>), dim3(grid), dim3(BLOCK), lds, st, p,
                         nfull, ntiles, slot0, fin);
      return true;
    }
  }
  if constexpr (MODE != MODE_ADAMW)
    hipLaunchKernelGGL((k_step<GT, J_T, MODE, BLOCK, ITERS, TABLE, GBAR, DEFER_T, COORD>), dim3(grid), dim3(BLOCK), lds, st, p,
                       nfull, ntiles, slot0);
  return false;
}

template <class GT, int MODE, bool TABLE, int BS, int IS, bool GBAR>
hipError_t launch_step_shape(const StepParams& p, int cls, int64_t nfull, int64_t ntiles, const Finish& fin, bool& ended,
                             hipStream_t st) {
  const bool long_class = cls == CLS_LONG;
  constexpr bool WRITES = (MODE != MODE_STATS) || GBAR;
  const bool gbar = MODE == MODE_STATS && p.gbar != nullptr;
  int64_t per_launch = launch_tiles(p.J, GT::ESIZE, MODE, gbar, cls, p.d, ntiles);
  if (WRITES && long_class) {
    // blocks that write per coordinate do so at the end of their lives: a launch holds whole generations of blocks
    // (as many as the chip runs at a time), so that all of them read together and write together
    int per_cu = 4;
    if constexpr (WRITES) {
#define NT_OCC(JJ)                                                                                          \
  case JJ:                                                                                                  \
    if constexpr (JJ * GT::ESIZE >= defer_row_bytes(MODE))                                                  \
      per_cu = blocks_per_cu<step_kernel<GT, JJ, MODE, NT_BLOCK_DEFER, NT_ITERS_DEFER, TABLE, true, true>(),       \
                             NT_BLOCK_DEFER>();                                                             \
    break;
      switch (p.J) {
        NT_OCC(2) NT_OCC(3) NT_OCC(4) NT_OCC(5) NT_OCC(6) NT_OCC(7) NT_OCC(8) NT_OCC(9)
        NT_OCC(10) NT_OCC(11) NT_OCC(12) NT_OCC(13) NT_OCC(14) NT_OCC(15) NT_OCC(16)
        default:
          per_cu = (p.J <= NT_FEW_ROWS)
                       ? blocks_per_cu<step_kernel<GT, 0, MODE, NT_BLOCK_FEW, NT_ITERS_FEW, TABLE, true>(), NT_BLOCK_FEW>()
                       : blocks_per_cu<step_kernel<GT, 0, MODE, NT_BLOCK_LARGE, NT_ITERS_LARGE, TABLE, true>(), NT_BLOCK_LARGE>();
      }
#undef NT_OCC
    }
    per_launch = (int64_t)cu_count() * per_cu * (p.J <= NT_JCHUNK ? NT_GENS_DEFER : NT_GENS_LARGE);
    if (per_launch > ntiles) per_launch = ntiles;
  }
  // AdamW only runs its launches from the last slots to the first: the launch with slot 0 writes the result (k_step_end), and
  // no result is to precede an update that has yet to be launched.  (Asking in the kernel for the last slot instead takes
  // scalar registers that the deferred kernels over pointer tables do not have: they would need scratch memory.)
  if (per_launch > NT_MAX_GRID) per_launch = NT_MAX_GRID;
  const int64_t runs = (ntiles + per_launch - 1) / per_launch;
  for (int64_t run = 0; run < runs; ++run) {
    const int64_t slot0 = (MODE == MODE_ADAMW ? runs - 1 - run : run) * per_launch;
    const unsigned grid = (unsigned)(ntiles - slot0 < per_launch ? ntiles - slot0 : per_launch);
#define NT_ARGS p, nfull, ntiles, slot0, grid, fin, st
#define NT_CASE(JJ)                                                                                             \
  case JJ:                                                                                                      \
    if constexpr (WRITES && JJ * GT::ESIZE >= defer_row_bytes(MODE)) {                                          \
      if (long_class) {                                                                                         \
        ended = launch_tiles_of<GT, JJ, MODE, NT_BLOCK_DEFER, NT_ITERS_DEFER, TABLE, true, false, true>(NT_ARGS); \
        break;                                                                                                  \
      }                                                                                                         \
    }                                                                                                           \
    if constexpr (plain_stats(GT::ESIZE, JJ, MODE, GBAR) || plain_coords(GT::ESIZE, JJ, MODE) > 0) {            \
      if (p.coord_thr < 0.f && (plain_stats(GT::ESIZE, JJ, MODE, GBAR) || p.d <= plain_coords(GT::ESIZE, JJ, MODE))) { \
        ended = launch_tiles_of<GT, JJ, MODE, BS, IS, TABLE, GBAR, GBAR, false, false>(NT_ARGS);                \
        break;                                                                                                  \
      }                                                                                                         \
    }                                                                                                           \
    ended = launch_tiles_of<GT, JJ, MODE, BS, IS, TABLE, GBAR, GBAR>(NT_ARGS);                                  \
    break;
    switch (p.J) {
      NT_CASE(2) NT_CASE(3) NT_CASE(4) NT_CASE(5) NT_CASE(6) NT_CASE(7) NT_CASE(8) NT_CASE(9)
      NT_CASE(10) NT_CASE(11) NT_CASE(12) NT_CASE(13) NT_CASE(14) NT_CASE(15) NT_CASE(16)
      default:
        if (cls == CLS_SHORT) {
          ended = launch_tiles_of<GT, 0, MODE, NT_BLOCK_MANY_TINY, NT_ITERS_MANY_TINY, TABLE, WRITES, true>(NT_ARGS);
        } else if (cls == CLS_TINY) {
          if constexpr (GT::ESIZE == 4)
            ended = launch_tiles_of<GT, 0, MODE, NT_SPLIT_TILE / NT_VEC, 1, TABLE, WRITES, true>(NT_ARGS);
          else if (p.J <= 2 * NT_MCHUNK)
            ended = launch_tiles_of<GT, NT_SPLIT + 2, MODE, 2 * NT_SPLIT_TILE / NT_VEC, 1, TABLE, WRITES, true>(NT_ARGS);
          else
            ended = launch_tiles_of<GT, NT_SPLIT + 4, MODE, 4 * NT_SPLIT_TILE / NT_VEC, 1, TABLE, WRITES, true>(NT_ARGS);
        } else if constexpr (MODE == MODE_STATS && !GBAR) {
          ended = launch_tiles_of<GT, 0, MODE, NT_BLOCK_LARGE_STATS, NT_ITERS_LARGE_STATS, TABLE, false, !TABLE>(NT_ARGS);
        } else {
          if (!long_class)
            ended = launch_tiles_of<GT, 0, MODE, NT_BLOCK_MANY_SHORT, NT_ITERS_MANY_SHORT, TABLE, true, !TABLE>(NT_ARGS);
          else if (p.J <= NT_FEW_ROWS)
            ended = launch_tiles_of<GT, 0, MODE, NT_BLOCK_FEW, NT_ITERS_FEW, TABLE, true, false>(NT_ARGS);
          else
            ended = launch_tiles_of<GT, 0, MODE, NT_BLOCK_LARGE, NT_ITERS_LARGE, TABLE, true, false>(NT_ARGS);
        }
    }
#undef NT_ARGS
#undef NT_CASE
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// picks the launch class (block size, sweeps per tile) that tile_cfg() describes
template <class GT, int MODE, bool TABLE>
hipError_t launch_step(const StepParams& p, int cls, int64_t nfull, int64_t ntiles, const Finish& fin, bool& ended,
                       hipStream_t st) {
  if constexpr (MODE == MODE_STATS) {
    // read-only statistics over a short vector borrow the kernels that can also store gbar (there is none to store)
    if (p.gbar || (cls == CLS_SHORT && p.J <= NT_JCHUNK))
      return launch_step_shape<GT, MODE, TABLE, NT_BLOCK_STATS_GBAR, NT_ITERS_STATS_GBAR, true>(p, cls, nfull, ntiles,
                                                                                                 fin, ended, st);
    return launch_step_shape<GT, MODE, TABLE, NT_BLOCK_STATS, NT_ITERS_STATS, false>(p, cls, nfull, ntiles, fin, ended, st);
  } else if constexpr (MODE == MODE_ADAMW) {
    return launch_step_shape<GT, MODE, TABLE, NT_BLOCK_ADAMW, NT_ITERS_ADAMW, true>(p, cls, nfull, ntiles, fin, ended, st);
  } else {
    return launch_step_shape<GT, MODE, TABLE, NT_BLOCK, NT_ITERS, true>(p, cls, nfull, ntiles, fin, ended, st);
  }
}

template <class GT, bool TABLE>
hipError_t launch_step_mode(int mode, const StepParams& p, int cls, int64_t nfull, int64_t ntiles, const Finish& fin,
                            bool& ended, hipStream_t st) {
  switch (mode) {
    case MODE_FULL: return launch_step<GT, MODE_FULL, TABLE>(p, cls, nfull, ntiles, fin, ended, st);
    case MODE_STATS: return launch_step<GT, MODE_STATS, TABLE>(p, cls, nfull, ntiles, fin, ended, st);
    default: return launch_step<GT, MODE_ADAMW, TABLE>(p, cls, nfull, ntiles, fin, ended, st);
  }
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace

extern "C" {

int64_t normtest_tile_coords(int64_t J) { return J >= 2 ? NT_TILE_MAX : 0; }

// Bytes of the record, the tile partials and the group partials: what every call needs.
static size_t partials_bytes(int64_t J, int64_t d) {
  const int64_t tc = min_tile_coords(J);
  int64_t ntiles = (d + tc - 1) / tc;
  if (J > NT_JCHUNK) {   // never less than a shorter vector takes
    const int64_t small = ((d < NT_SPLIT_COORDS ? d : NT_SPLIT_COORDS) + NT_SPLIT_TILE - 1) / NT_SPLIT_TILE;
    if (small > ntiles) ntiles = small;
  }
  const int64_t n = ntiles > 0 ? ntiles : 1;
  return (size_t)(NT_WS_HEADER + n * NT_NV + most_groups(ntiles) * 2 * NT_NV) * sizeof(double);
}

size_t normtest_workspace_bytes(int64_t J, int64_t d) {
  if (J < 2 || d < 0) return 0;
  return partials_bytes(J, d);
}

// dtype and flags do not change the size (they did while many-row steps kept gbar in the workspace)
size_t normtest_workspace_bytes_for(nt_dtype gdtype, int64_t J, int64_t d, uint32_t flags) {
  (void)flags;
  if (J < 2 || d < 0 || (gdtype != NT_F32 && gdtype != NT_BF16)) return 0;
  return partials_bytes(J, d);
}

// AdamW constants in fp64 on the host, rounded once to fp32.
static void fill_adamw_params(StepParams& p, const nt_hyper* hyper) {
  const double bc1 = 1.0 - std::pow(hyper->beta1, (double)hyper->step);
  const double bc2 = 1.0 - std::pow(hyper->beta2, (double)hyper->step);
  p.beta1 = (float)hyper->beta1;
  p.omb1 = (float)(1.0 - hyper->beta1);
  p.beta2 = (float)hyper->beta2;
  p.omb2 = (float)(1.0 - hyper->beta2);
  p.decay = (float)(1.0 - hyper->lr * hyper->weight_decay);
  p.step_size = (float)(hyper->lr / bc1);
  p.inv_sqrt_bc2 = (float)(1.0 / std::sqrt(bc2));
  p.eps = (float)hyper->eps;
}

// Validation shared by normtest_step and normtest_step_clipped; `flags` are the flags the kernels
// will run with.  Nothing is enqueued here.
static int check_step_args(const void* grads, nt_dtype gdtype, int64_t J, int64_t d, int64_t ld, const float* w,
                           const float* m, const float* v, const float* gbar_out, uint32_t flags,
                           const nt_hyper* hyper, const nt_shard_info* shard, const void* workspace,
                           size_t workspace_bytes, const nt_result* result_dev) {
  if (gdtype != NT_F32 && gdtype != NT_BF16) return NT_ERR_UNSUPPORTED;
  if (J < 2 || J > (1 << 20) || d < 0 || ld < d) return NT_ERR_BAD_ARG;
  if (!hyper_ok(hyper, J) || !result_dev || !workspace) return NT_ERR_BAD_ARG;
  if (((uintptr_t)result_dev & 7u) || ((uintptr_t)workspace & 7u)) return NT_ERR_BAD_ARG;
  if (d > 0 && !grads) return NT_ERR_BAD_ARG;
  if (d > 0 && (flags & NT_DO_ADAMW) && (!w || !m || !v)) return NT_ERR_BAD_ARG;
  if (d > 0 && (flags & NT_WRITE_GBAR) && !gbar_out) return NT_ERR_BAD_ARG;
  const int esize = gdtype == NT_F32 ? 4 : 2;
  if (((uintptr_t)grads & (uintptr_t)(esize - 1)) || ((uintptr_t)w & 3u) || ((uintptr_t)m & 3u) ||
      ((uintptr_t)v & 3u) || ((flags & NT_WRITE_GBAR) && ((uintptr_t)gbar_out & 3u)))
    return NT_ERR_BAD_ARG;
  if (shard) {
    if (shard->num_shards < 1 || shard->shard_id < 0 || shard->shard_id >= shard->num_shards ||
        shard->shard_offset < 0 || shard->d_global < 0 || shard->shard_offset + d > shard->d_global)
      return NT_ERR_BAD_ARG;
  }
  if (workspace_bytes < normtest_workspace_bytes_for(gdtype, J, d, flags)) return NT_ERR_WORKSPACE_TOO_SMALL;
  return NT_OK;
}

// Address of this device's copy of `scratch` or `tickets`, looked up once per device (the array's name is only a host-side
// handle of the symbol; kernels, copies and fills take this pointer).
typedef void* PerDevice[64];
static int device_address(const void* symbol, PerDevice& cached, void** out, int* device = nullptr) {
  int dev = 0;
  const hipError_t e0 = hipGetDevice(&dev);
  if (e0 != hipSuccess) return hip_code(e0);
  if (dev < 0 || dev >= 64) return NT_ERR_UNSUPPORTED;
  void* ptr = __atomic_load_n(&cached[dev], __ATOMIC_ACQUIRE);
  if (!ptr) {
    const hipError_t e = hipGetSymbolAddress(&ptr, symbol);
    if (e != hipSuccess) return hip_code(e);
    if (!ptr) return NT_ERR_UNSUPPORTED;
    __atomic_store_n(&cached[dev], ptr, __ATOMIC_RELEASE);
  }
  *out = ptr;
  if (device) *device = dev;
  return NT_OK;
}

// Whether a launch on st runs on the current device: the null stream and its two named forms do, other streams have a device of
// their own.
static bool on_current_device(hipStream_t st) {
  if (st == nullptr || st == hipStreamLegacy || st == hipStreamPerThread) return true;
  int current = 0;
  hipDevice_t own = 0;
  return hipGetDevice(&current) == hipSuccess && hipStreamGetDevice(st, &own) == hipSuccess && own == current;
}

// A stream's place among the counters, or -1 where there is none left near its hash: the step then takes a reduction kernel.  A place
// is kept until the process ends.  It passes to a stream that is made with the handle of one that was destroyed, whose work has ended
// then: HIP lets nobody count on work that a stream was destroyed with.  hipStreamPerThread is another stream in every thread.
static int stream_slot(int dev, hipStream_t st) {
  static uint64_t taken[NT_STREAMS];
  static thread_local char own;
  const uint64_t handle = (uint64_t)(uintptr_t)(st == hipStreamPerThread ? (const void*)&own : (const void*)st);
  const uint64_t key = (handle << 7) + 2 * (uint64_t)dev + 1;   // dev < 64
  const uint64_t at = key * 0x9e3779b97f4a7c15ull >> 32;
  for (uint64_t k = 0; k < 16; ++k) {
    uint64_t* place = &taken[(at + k) % NT_STREAMS];
    uint64_t who = __atomic_load_n(place, __ATOMIC_RELAXED);
    if (who == 0) __atomic_compare_exchange_n(place, &who, key, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED);   // who: 0, or who was faster
    if (who == 0 || who == key) return (int)(place - taken);
  }
  return -1;
}

// The counter of this stream, or false where there is none for this launch: a graph under capture would keep it and
// replay beside a later call on the stream, and the blocks of a launch on another device would count themselves in
// memory that is not theirs.
static bool stream_ticket(hipStream_t st, uint32_t** out) {
  static PerDevice cached = {nullptr};
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  void* base = nullptr;
  int dev = 0;
  if (hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone || !on_current_device(st) ||
      device_address(HIP_SYMBOL(tickets), cached, &base, &dev) != NT_OK) {
    (void)hipGetLastError();
    return false;
  }
  const int slot = stream_slot(dev, st);
  if (slot < 0) return false;
  *out = (uint32_t*)base + slot;
  return true;
}

// Enqueue the streaming kernel and the reduction/decision kernels.  Arguments are already validated.
// `table`: grads is a device array of J row pointers instead of the first row of a strided matrix.
// `d_whole`: length of the vector these d coordinates are a part of (d itself for a call that stands alone).
static int enqueue_step(const void* grads, bool table, nt_dtype gdtype, int64_t J, int64_t d, int64_t d_whole,
                        int64_t ld, float* w, float* m, float* v, float* gbar_out, uint32_t flags, const nt_hyper* hyper,
                        double max_norm, void* workspace, nt_result* result_dev, hipStream_t st) {
  const int esize = gdtype == NT_F32 ? 4 : 2;
  const int mode = (flags & NT_DO_STATS) ? ((flags & NT_DO_ADAMW) ? MODE_FULL : MODE_STATS) : MODE_ADAMW;
  const int cls = launch_class(J, esize, mode, (flags & NT_WRITE_GBAR) != 0, d_whole);
  const int64_t tc = tile_cfg(J, esize, mode, (flags & NT_WRITE_GBAR) != 0, d_whole).coords();
  const int64_t ntiles = (d + tc - 1) / tc;

  StepParams p;
  std::memset(&p, 0, sizeof(p));
  p.grads = grads;
  p.ld = ld;
  p.d = d;
  p.J = (int)J;
  p.w = w;
  p.m = m;
  p.v = v;
  p.gbar = (flags & NT_WRITE_GBAR) ? gbar_out : nullptr;
  p.partials = (double*)workspace + NT_WS_HEADER;
  p.inv_J = 1.0 / (double)J;
  if (flags & NT_DO_ADAMW) fill_adamw_params(p, hyper);
  p.coord_thr = (flags & NT_COORD_TEST)
                    ? (float)(hyper->eta * hyper->eta * (double)hyper->b_k * (double)(J - hyper->ddof))
                    : -1.0f;

  DecideParams q;
  q.J = J;
  q.eta = hyper->eta;
  q.max_norm = max_norm;
  q.b_k = hyper->b_k;
  q.b_max = hyper->b_max;
  q.round_to = hyper->round_to;
  q.ddof = hyper->ddof;
  q.flags = flags;
  const bool two_level = (flags & NT_DO_STATS) && ntiles > NT_DIRECT_TILES;
  const int64_t ngroups = two_level ? (ntiles + group_tiles(ntiles) - 1) / group_tiles(ntiles) : 0;
  WsHeader hdr;
  std::memset(&hdr, 0, sizeof(hdr));
  hdr.magic = NT_WS_MAGIC;
  hdr.tile_coords = tc;
  hdr.ntiles = ntiles;
  hdr.ngroups = ngroups;
  hdr.d = d;
  hdr.J = J;
  hdr.gdtype = (int32_t)gdtype;
  hdr.has_stats = (flags & NT_DO_STATS) ? 1 : 0;
  hdr.coord_thr = (double)p.coord_thr;
  hdr.q = q;
  WsRecord record;
  std::memcpy(&record, &hdr, sizeof(record));
  WsRecord* hdr_out = (WsRecord*)workspace;
  bool ended = false;   // the result has been left to the step's own kernel
  if (ntiles > 0) {
    Finish fin;
    std::memset(&fin, 0, sizeof(fin));
    // no sums, one partial that is the total, or few enough for the last block: launch_tiles_of has the kernels
    const int64_t most = J > NT_JCHUNK ? (cls == CLS_TINY ? NT_TICKET_TILES : NT_TICKET_TILES_MANY)
                                       : mode == MODE_STATS ? NT_TICKET_TILES_STATS : NT_TICKET_TILES;
    if (mode == MODE_ADAMW || ntiles == 1 || (ntiles <= most && stream_ticket(st, &fin.ticket))) {
      fin.q = q;
      fin.hdr = record;
      fin.hdr_out = hdr_out;
      fin.out = result_dev;
    }
    const int64_t nfull = d / tc;
    hipError_t e;
    if (table)
      e = (gdtype == NT_F32) ? launch_step_mode<F32, true>(mode, p, cls, nfull, ntiles, fin, ended, st)
                             : launch_step_mode<BF16, true>(mode, p, cls, nfull, ntiles, fin, ended, st);
    else
      e = (gdtype == NT_F32) ? launch_step_mode<F32, false>(mode, p, cls, nfull, ntiles, fin, ended, st)
                             : launch_step_mode<BF16, false>(mode, p, cls, nfull, ntiles, fin, ended, st);
    if (e != hipSuccess) return hip_code(e);
  }
  if (ended) return NT_OK;

  const double* partials = (const double*)workspace + NT_WS_HEADER;
  if (two_level)
    hipLaunchKernelGGL(k_reduce_end, dim3((unsigned)ngroups), dim3(NT_FIN_THREADS), 0, st, partials, ntiles,
                       (double*)workspace + NT_WS_HEADER + NT_NV * ntiles, q, result_dev, record, hdr_out);
  else
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(NT_FIN_THREADS), 0, st, partials, ntiles, q, result_dev, record, hdr_out);
  return hip_code(hipGetLastError());
}

// Enqueue AdamW on scale * gbar (phase 2 of the clipped variant).  Arguments are already validated.
static int enqueue_adamw_gbar(const float* gbar, int64_t d, float* w, float* m, float* v, const nt_hyper* hyper,
                              double grad_scale, const nt_result* result_dev, hipStream_t st) {
  if (d == 0) return NT_OK;
  StepParams p;
  std::memset(&p, 0, sizeof(p));
  p.d = d;
  p.w = w;
  p.m = m;
  p.v = v;
  fill_adamw_params(p, hyper);
  const int64_t per_block = (int64_t)NT_AUX_BLOCK * NT_VEC;
  const int64_t nblocks = (d + per_block - 1) / per_block;
  // in runs of blocks, like the step kernel (see NT_CHUNK_FULL)
  const int64_t per_launch = NT_CHUNK_ADAMW_GBAR / per_block;
  for (int64_t b0 = 0; b0 < nblocks; b0 += per_launch) {
    const int64_t grid = (nblocks - b0 < per_launch) ? nblocks - b0 : per_launch;
    hipLaunchKernelGGL(k_adamw_gbar, dim3((unsigned)grid), dim3(NT_AUX_BLOCK), d >= (1ll << 25) ? NT_ONE_BLOCK_LDS : 0, st, p,
                       gbar, (float)grad_scale, result_dev, b0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_code(e);
  }
  return NT_OK;
}

// Length of the vector a call's d coordinates belong to: what the caller's shard record says, else d.
inline int64_t whole_length(int64_t d, const nt_shard_info* shard) {
  return (shard && shard->d_global > d) ? shard->d_global : d;
}

// The step as the caller's flags describe it, always one pass (NT_ONE_PASS, which once kept many-row steps from
// being split into two passes, is accepted and changes nothing).
static int enqueue_step_routed(const void* grads, bool table, nt_dtype gdtype, int64_t J, int64_t d,
                               const nt_shard_info* shard, int64_t ld, float* w, float* m, float* v, float* gbar_out,
                               const nt_hyper* hyper, void* workspace, nt_result* result_dev, hipStream_t st) {
  return enqueue_step(grads, table, gdtype, J, d, whole_length(d, shard), ld, w, m, v, gbar_out, hyper->flags, hyper, 0.0,
                      workspace, result_dev, st);
}

int normtest_step(const void* grads, nt_dtype gdtype, int64_t J, int64_t d, int64_t ld, float* w, float* m,
                  float* v, float* gbar_out, const nt_hyper* hyper, const nt_shard_info* shard, void* workspace,
                  size_t workspace_bytes, nt_result* result_dev, void* hip_stream) {
  if (!hyper) return NT_ERR_BAD_ARG;
  const int rc = check_step_args(grads, gdtype, J, d, ld, w, m, v, gbar_out, hyper->flags, hyper, shard, workspace,
                                 workspace_bytes, result_dev);
  if (rc != NT_OK) return rc;
  return enqueue_step_routed(grads, false, gdtype, J, d, shard, ld, w, m, v, gbar_out, hyper, workspace, result_dev,
                             (hipStream_t)hip_stream);
}

int normtest_step_rows(const void* const* grad_rows_dev, nt_dtype gdtype, int64_t J, int64_t d, float* w, float* m,
                       float* v, float* gbar_out, const nt_hyper* hyper, const nt_shard_info* shard, void* workspace,
                       size_t workspace_bytes, nt_result* result_dev, void* hip_stream) {
  if (!hyper || ((uintptr_t)grad_rows_dev & 7u)) return NT_ERR_BAD_ARG;
  // the table stands in for the matrix; its entries cannot be inspected from the host
  const int rc = check_step_args(grad_rows_dev, gdtype, J, d, d, w, m, v, gbar_out, hyper->flags, hyper, shard,
                                 workspace, workspace_bytes, result_dev);
  if (rc != NT_OK) return rc;
  return enqueue_step_routed(grad_rows_dev, true, gdtype, J, d, shard, d, w, m, v, gbar_out, hyper, workspace, result_dev,
                             (hipStream_t)hip_stream);
}

int64_t normtest_static_max_coords(int64_t J) {
  if (J < 2 || J > (1 << 20)) return 0;
  // largest d whose record, tile partials and group partials fit: partials_bytes is monotone in d
  int64_t lo = 0, hi = (int64_t)1 << 40;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo + 1) / 2;
    if (partials_bytes(J, mid) <= NT_SCRATCH_BYTES) lo = mid; else hi = mid - 1;
  }
  return lo;
}

int normtest_step_static(const void* grads, nt_dtype gdtype, int64_t J, int64_t d, int64_t ld, float* w, float* m,
                         float* v, float* gbar_out, const nt_hyper* hyper, const nt_shard_info* shard,
                         nt_result* result_dev, void* hip_stream) {
  if (!hyper) return NT_ERR_BAD_ARG;
  if (J >= 2 && J <= (1 << 20) && d > normtest_static_max_coords(J)) return NT_ERR_TOO_LARGE;
  nt_hyper hy = *hyper;
  // validate with a stand-in for the workspace (any non-null, aligned address: nothing is enqueued here)
  const int rc = check_step_args(grads, gdtype, J, d, ld, w, m, v, gbar_out, hy.flags, &hy, shard, (const void*)256,
                                 (size_t)-1, result_dev);
  if (rc != NT_OK) return rc;
  static PerDevice cached = {nullptr};
  void* ws = nullptr;
  const int rs = device_address(HIP_SYMBOL(scratch), cached, &ws);
  if (rs != NT_OK) return rs;
  return enqueue_step_routed(grads, false, gdtype, J, d, shard, ld, w, m, v, gbar_out, &hy, ws, result_dev,
                             (hipStream_t)hip_stream);
}

int normtest_step_clipped(const void* grads, nt_dtype gdtype, int64_t J, int64_t d, int64_t ld, float* w, float* m,
                          float* v, float* gbar_buf, double max_norm, const nt_hyper* hyper,
                          const nt_shard_info* shard, void* workspace, size_t workspace_bytes, nt_result* result_dev,
                          void* hip_stream) {
  if (!hyper || std::isnan(max_norm)) return NT_ERR_BAD_ARG;
  const uint32_t need = NT_DO_STATS | NT_DO_ADAMW;
  if ((hyper->flags & need) != need || (hyper->flags & NT_PARTIAL)) return NT_ERR_BAD_ARG;
  // validate as the fused step with the mean written out (this also checks w, m, v and the AdamW scalars)
  const int rc = check_step_args(grads, gdtype, J, d, ld, w, m, v, gbar_buf, hyper->flags | NT_WRITE_GBAR, hyper,
                                 shard, workspace, workspace_bytes, result_dev);
  if (rc != NT_OK) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  const int rc1 = enqueue_step(grads, false, gdtype, J, d, whole_length(d, shard), ld, nullptr, nullptr, nullptr, gbar_buf,
                               NT_DO_STATS | NT_WRITE_GBAR | (hyper->flags & NT_COORD_TEST), hyper, max_norm, workspace,
                               result_dev, st);
  if (rc1 != NT_OK) return rc1;
  return enqueue_adamw_gbar(gbar_buf, d, w, m, v, hyper, 1.0, result_dev, st);
}

int normtest_layer_stats(const void* grads, int rows_are_table, nt_dtype gdtype, int64_t J, int64_t d, int64_t ld,
                         const int64_t* layer_offsets_dev, int32_t L, const void* workspace,
                         nt_layer_stats* layers_dev, void* hip_stream) {
  if (gdtype != NT_F32 && gdtype != NT_BF16) return NT_ERR_UNSUPPORTED;
  if (J < 2 || J > (1 << 20) || d < 0 || (!rows_are_table && ld < d)) return NT_ERR_BAD_ARG;
  if (L < 1 || L > (1 << 24) || !layer_offsets_dev || !workspace || !layers_dev) return NT_ERR_BAD_ARG;
  if (((uintptr_t)layer_offsets_dev & 7u) || ((uintptr_t)workspace & 7u) || ((uintptr_t)layers_dev & 7u))
    return NT_ERR_BAD_ARG;
  if (d > 0 && !grads) return NT_ERR_BAD_ARG;
  const int esize = gdtype == NT_F32 ? 4 : 2;
  if ((uintptr_t)grads & (uintptr_t)(rows_are_table ? 7 : esize - 1)) return NT_ERR_BAD_ARG;
  StepParams p;
  std::memset(&p, 0, sizeof(p));
  p.grads = grads;
  p.ld = rows_are_table ? d : ld;
  p.d = d;
  p.J = (int)J;
  p.inv_J = 1.0 / (double)J;
  p.coord_thr = -1.0f;  // the kernel takes the threshold of the recorded step
  hipStream_t st = (hipStream_t)hip_stream;
  const double* ws = (const double*)workspace;
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(L), dim3(threads), 0, st, p, layer_offsets_dev, ws, layers_dev);
  };
  const bool table = rows_are_table != 0, many = J > NT_JCHUNK;
#define NT_LAYERS(GT, TABLE, MANY) \
  if (table == TABLE && many == MANY) launch(k_layer_stats<GT, TABLE, MANY>, layer_threads<GT, MANY>());
  if (gdtype == NT_F32) {
    NT_LAYERS(F32, false, false) NT_LAYERS(F32, false, true) NT_LAYERS(F32, true, false) NT_LAYERS(F32, true, true)
  } else {
    NT_LAYERS(BF16, false, false) NT_LAYERS(BF16, false, true) NT_LAYERS(BF16, true, false) NT_LAYERS(BF16, true, true)
  }
#undef NT_LAYERS
  return hip_code(hipGetLastError());
}

int normtest_adamw_gbar(const float* gbar, int64_t d, float* w, float* m, float* v, const nt_hyper* hyper,
                        double grad_scale, const nt_result* result_dev, void* hip_stream) {
  if (!hyper || d < 0 || !std::isfinite(grad_scale)) return NT_ERR_BAD_ARG;
  if (hyper->step < 1 || !(hyper->lr >= 0.0) || !std::isfinite(hyper->lr) ||
      !(hyper->beta1 >= 0.0 && hyper->beta1 < 1.0) || !(hyper->beta2 >= 0.0 && hyper->beta2 < 1.0) ||
      !(hyper->eps >= 0.0) || !std::isfinite(hyper->eps) || !(hyper->weight_decay >= 0.0) ||
      !std::isfinite(hyper->weight_decay))
    return NT_ERR_BAD_ARG;
  if (d > 0 && (!gbar || !w || !m || !v)) return NT_ERR_BAD_ARG;
  if (((uintptr_t)gbar & 3u) || ((uintptr_t)w & 3u) || ((uintptr_t)m & 3u) || ((uintptr_t)v & 3u) ||
      ((uintptr_t)result_dev & 7u))
    return NT_ERR_BAD_ARG;
  return enqueue_adamw_gbar(gbar, d, w, m, v, hyper, grad_scale, result_dev, (hipStream_t)hip_stream);
}

double normtest_clip_coef(double gbar_sq, double max_norm) { return clip_coef(gbar_sq, max_norm); }

int normtest_resplit(int64_t b, int64_t J, int64_t accum_base, int64_t micro_max, int64_t* micro, int64_t* accum,
                     int64_t* global_batch) {
  if (b < 1 || J < 1 || accum_base < 1 || micro_max < 1 || !micro || !accum || !global_batch) return NT_ERR_BAD_ARG;
  // samples each worker must see, accumulation steps needed at the largest micro-batch, never below the base
  const int64_t per_worker = (b + J - 1) / J;
  int64_t steps = (per_worker + micro_max - 1) / micro_max;
  if (steps < accum_base) steps = accum_base;
  const int64_t chunk = J * steps;
  *micro = (b + chunk - 1) / chunk;
  *accum = steps;
  *global_batch = chunk * *micro;
  return NT_OK;
}

uint32_t normtest_schedule_flags(int64_t step, int64_t test_interval, int64_t b_k, int64_t b_max, uint32_t flags) {
  if (step < 1 || test_interval < 1 || b_k < 1 || b_max < 0) return flags;
  const bool at_maximum = b_max > 0 && b_k >= b_max;
  const bool on_interval = (step - 1) % test_interval == 0;
  if (on_interval && !at_maximum) return flags;
  return flags & ~(uint32_t)(NT_DO_STATS | NT_PARTIAL | NT_COORD_TEST);
}

int normtest_combine(const nt_result* partials, int32_t n, int64_t J, const nt_hyper* hyper, nt_result* out) {
  if (!partials || !out || n < 1 || J < 2 || !hyper) return NT_ERR_BAD_ARG;
  if (!(hyper->eta > 0.0) || !std::isfinite(hyper->eta) || hyper->b_k < 1 || hyper->b_max < 0 ||
      hyper->round_to < 1 || hyper->round_to > NT_ROUND_TO_MAX || (hyper->ddof != 0 && hyper->ddof != 1) || J - hyper->ddof < 1)
    return NT_ERR_BAD_ARG;
  dd tot[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
  uint32_t status = 0;
  int64_t coord_fail = 0;  // the count is additive over shards; missing in one shard = missing in the total
  double coord_max = 0.0;  // the largest ratio over shards is the largest of the shards' values
  for (int32_t s = 0; s < n; ++s) {
    if (partials[s].status & NT_STATUS_NO_STATS) return NT_ERR_BAD_ARG;
    coord_fail = (coord_fail < 0 || partials[s].coord_fail < 0) ? -1 : coord_fail + partials[s].coord_fail;
    if (partials[s].coord_fail >= 0 && partials[s].coord_max_ratio > coord_max) coord_max = partials[s].coord_max_ratio;
    const dd a = {partials[s].A, partials[s].A_lo}, b = {partials[s].B, partials[s].B_lo},
             c = {partials[s].C, partials[s].C_lo};
    tot[0] = dd_add(tot[0], a);
    tot[1] = dd_add(tot[1], b);
    tot[2] = dd_add(tot[2], c);
    status |= partials[s].status & NT_STATUS_NONFINITE;
  }
  nt_result r;
  std::memset(&r, 0, sizeof(r));
  r.A = tot[0].hi; r.A_lo = tot[0].lo;
  r.B = tot[1].hi; r.B_lo = tot[1].lo;
  r.C = tot[2].hi; r.C_lo = tot[2].lo;
  if (status & NT_STATUS_NONFINITE) {
    // a non-finite low part would otherwise poison finite high parts; report the plain sums
    r.A = r.B = r.C = 0.0;
    for (int32_t s = 0; s < n; ++s) {
      r.A += partials[s].A;
      r.B += partials[s].B;
      r.C += partials[s].C;
    }
    r.A_lo = r.B_lo = r.C_lo = 0.0;
  }
  r.status = 0;
  DecideParams q;
  q.J = J;
  q.eta = hyper->eta;
  q.b_k = hyper->b_k;
  q.b_max = hyper->b_max;
  q.round_to = hyper->round_to;
  q.max_norm = 0.0;
  q.ddof = hyper->ddof;
  q.flags = NT_DO_STATS;
  decide(q, &r);
  r.coord_fail = coord_fail;
  r.coord_max_ratio = coord_fail < 0 ? -1.0 : coord_max;
  *out = r;
  return NT_OK;
}

int normtest_calib_copy(void* dst, const void* src, size_t bytes, void* hip_stream) {
  if (!dst || !src || !aligned16(dst) || !aligned16(src) || (bytes & 15u)) return NT_ERR_BAD_ARG;
  if (bytes == 0) return NT_OK;
  const int64_t n16 = (int64_t)(bytes / 16);
  const int64_t want = (n16 + NT_AUX_BLOCK - 1) / NT_AUX_BLOCK;
  const int64_t max_grid = (int64_t)cu_count() * NT_COPY_BLOCKS_PER_CU;
  const int grid = (int)(want < max_grid ? want : max_grid);
  hipLaunchKernelGGL(k_copy16, dim3(grid), dim3(NT_AUX_BLOCK), 0, (hipStream_t)hip_stream, (f32x4*)dst,
                     (const u32x4*)src, n16);
  return hip_code(hipGetLastError());
}

int normtest_calib_streams(void* buf, size_t buf_bytes, int64_t coords, int row_reads, int reads, int writes, int rmw,
                           int64_t launch_coords, void* hip_stream) {
  if (!buf || !aligned16(buf) || coords < 0 || (coords & 3) || row_reads < 0 || reads < 0 || writes < 0 ||
      launch_coords < 0 || (launch_coords & 3))
    return NT_ERR_BAD_ARG;
  if (row_reads > NT_CALIB_MAX_R8 || reads > NT_CALIB_MAX_R16 || writes > NT_CALIB_MAX_W || row_reads + reads + writes == 0)
    return NT_ERR_UNSUPPORTED;
  // streams sit one after the other: row-like ones of 2 bytes per coordinate first, then those of 4
  const size_t row_bytes = (((size_t)coords * 2 + 255u) & ~(size_t)255u), vec_bytes = (((size_t)coords * 4 + 255u) & ~(size_t)255u);
  const size_t need = row_bytes * (size_t)row_reads + vec_bytes * (size_t)(reads + writes) + 16;
  if (buf_bytes < need) return NT_ERR_WORKSPACE_TOO_SMALL;
  if (coords == 0) return NT_OK;
  CalibStreams s;
  std::memset(&s, 0, sizeof(s));
  char* at = (char*)buf;
  for (int k = 0; k < row_reads; ++k, at += row_bytes) s.r8[k] = at;
  for (int k = 0; k < reads; ++k, at += vec_bytes) s.r16[k] = at;
  for (int k = 0; k < writes; ++k, at += vec_bytes) s.w[k] = at;
  s.sink = (uint32_t*)at;
  const int64_t ngroups = coords / 4;
  // like the step kernel, in launches over runs of consecutive coordinates (whole blocks) if the caller says so
  const int64_t per_block = NT_AUX_BLOCK;
  int64_t per_launch = launch_coords > 0 ? launch_coords / 4 / per_block * per_block : ngroups;
  if (per_launch < per_block) per_launch = per_block;
  const int64_t max_grid = (int64_t)cu_count() * NT_COPY_BLOCKS_PER_CU;
  hipStream_t st = (hipStream_t)hip_stream;
  bool found = false;
#define NT_CALIB(R8, R16, W, RMW)                                                                                  \
  if (!found && row_reads == R8 && reads == R16 && writes == W && (rmw != 0) == RMW) {                              \
    for (int64_t g0 = 0; g0 < ngroups; g0 += per_launch) {                                                         \
      const int64_t g1 = (ngroups - g0 < per_launch) ? ngroups : g0 + per_launch;                                  \
      const int64_t want = (g1 - g0 + per_block - 1) / per_block;                                                  \
      const int grid = (int)(want < max_grid ? want : max_grid);                                                   \
      hipLaunchKernelGGL((k_calib_streams<R8, R16, W, RMW>), dim3(grid), dim3(NT_AUX_BLOCK), 0, st, s, g0, g1);    \
    }                                                                                                              \
    found = true;                                                                                                  \
  }
#define NT_CALIB_ROW(R16) NT_CALIB(0, R16, 0, false) NT_CALIB(0, R16, 1, false) NT_CALIB(0, R16, 2, false) NT_CALIB(0, R16, 3, false)
  // the matrix of read streams x written streams ...
  NT_CALIB(0, 0, 1, false) NT_CALIB(0, 0, 2, false) NT_CALIB(0, 0, 3, false)
  NT_CALIB_ROW(1) NT_CALIB_ROW(2) NT_CALIB_ROW(4) NT_CALIB_ROW(8) NT_CALIB_ROW(11)
  // ... in-place updates alone ...
  NT_CALIB(0, 0, 1, true) NT_CALIB(0, 0, 3, true)
  // ... and the traffic of the step itself: J row reads with three in-place fp32 arrays, rows alone, and the same
  // bytes with the results going to separate arrays
  NT_CALIB(4, 0, 3, true) NT_CALIB(8, 0, 3, true) NT_CALIB(16, 0, 3, true)
  NT_CALIB(4, 0, 0, false) NT_CALIB(8, 0, 0, false) NT_CALIB(16, 0, 0, false)
  NT_CALIB(8, 0, 1, false) NT_CALIB(8, 3, 3, false)
#undef NT_CALIB_ROW
#undef NT_CALIB
  if (!found) return NT_ERR_UNSUPPORTED;
  return hip_code(hipGetLastError());
}

const char* normtest_strerror(int code) {
  switch (code) {
    case NT_OK: return "success";
    case NT_ERR_BAD_ARG: return "bad argument (null or misaligned pointer, J < 2, d < 0, ld < d, or invalid hyper-parameters)";
    case NT_ERR_UNSUPPORTED: return "unsupported gradient dtype";
    case NT_ERR_WORKSPACE_TOO_SMALL: return "workspace smaller than normtest_workspace_bytes(J, d)";
    case NT_ERR_TOO_LARGE: return "d beyond normtest_static_max_coords(J): the built-in scratch cannot hold the partial sums";
    default: break;
  }
  if (code <= NT_ERR_HIP_BASE) return hipGetErrorString((hipError_t)(NT_ERR_HIP_BASE - code));
  return "unknown error code";
}

}  // extern "C"
