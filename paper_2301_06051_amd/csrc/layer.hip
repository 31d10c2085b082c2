// dsvt_set_attention / dsvt_block: one DSVT layer per kernel launch on gfx950 (Sec. 3.2 Eq. 4-5;
// appendix "Network Architecture").
//
// k_layer: a workgroup owns a run of consecutive sets (a "tile" of at most 96 rows).  It takes the
// sets' distinct voxels -- from the tile descriptor the partition wrote, or, without a work list, by
// keeping the first occurrence of every voxel in the sets' slot rows (repeats are adjacent, Eq. 3 is
// monotone) -- and gathers those voxels' features into an LDS tile: the tau x C tiles of Eq. (4)
// with the repeated rows squeezed out, since a masked repeat contributes nothing as a key and its
// query row would be thrown away.  Q/K/V projection, per-(set, head) softmax(QK^T + PE)V,
// output projection, residual + LayerNorm, the MLP and the second residual + LayerNorm all run
// on that tile in LDS and registers; the rows then go straight back to the voxels' rows of the
// output (every voxel is in exactly one set, Thm A.2-A.3), so a layer reads and writes [N, C] once.
#include "common.h"
#include "mma.h"
#include "phase_clock.h"
#include <cfloat>

namespace {

constexpr int kTauMax = 96;                     // a set's distinct voxels must fit one tile
constexpr int kMaxSets = kRowsMax / 4;           // every set takes at least 4 rows of a tile
constexpr int kRowsPad = kRowsMax + 16;          // per-row arrays are read 4 at a time up to 15 rows past a set's end
constexpr int kHdrWords = 64;                   // header of a tile descriptor: rows, sets, the sets' first rows, their distinct voxels
constexpr int kHdrR0 = 2, kHdrNu = kHdrR0 + kMaxSets;
constexpr int kRelRow = 16;                      // bytes of a position table's row: four heads
constexpr int kSetWords = 32;                   // set table of the attention phase, see set_word()
static_assert(kMaxSets <= kSetWords && kHdrNu + kSetWords <= kHdrWords, "a word per set");
// Sets per workgroup when no tile list is given.
__host__ __device__ constexpr int fixed_sets(int tau) { return tau <= kRowsMax / 2 ? 2 : 1; }
// The sets a kernel is instantiated for: of up to three key tiles (48 voxels), or of up to six (96), these last also in
// a form of fewer registers.
enum SetSize { kSets48, kSets96, kSets96Slim };
// A set of up to 3 key tiles (48 voxels) is split into items of half of the heads each.  A larger one's logits and positional terms
// take more registers, and what bounds its items is the fetching of the terms, a load of the compute unit's memory pipe per key and
// query tile whatever its width: C = 128 takes four heads an item, 32 keys at a time (attn_item()), the other shapes two heads and all keys (C = 192
// spills 40 registers and more with four; C = 64 has four heads), kSets96Slim one, and so does C = 192 with repeats counted as keys.  (There two spilled
// when the line was drawn.  With the sums as they are now they do not, and a block of 20,000 voxels, 30 x 30 windows, sets of up to 90, takes 81.3 us where one
// head takes 98.4, of 30,000 in 24 x 24 windows, sets of up to 60, 84.4 where it takes 89.7: not drawn anew yet.)  C = 128, two heads -> four: the same two blocks
// 63.3 -> 58.5 us and 56.4 -> 54.5; attention of a tile of 70 rows 16.3 -> 12.0 k clocks.  At most one set of a tile is that large, so a tile has
// at most 8 * 6 + 2 * (3 + 11) = 76 items.
__host__ __device__ constexpr int big_heads(int C, bool dup, SetSize sz) { return sz == kSets96Slim || (C == 192 && dup) ? 1 : C == 128 ? 4 : 2; }
__host__ __device__ constexpr int item_groups(int kts, int heads, int big) { return kts <= 3 ? 2 : heads / big; }
// A tile whose items leave half of the wavefronts without one -- a set or two: sparse frames -- gets items of a quarter of
// the heads (sets of up to three key tiles; a larger one makes 8 to 12 items at C = 128 and 64, 16 and more at C = 192).  An item's heads go through its
// steps together, so half as many of them take little less than all.  Never split -> so: pass of 3,001 pillars 135.3 -> 134.4 us (attention
// of its tiles of 24 rows 4.8 k of 26.6 k clocks), one block of 2,000 voxels in fp32 47.4 -> 47.1; frames of full tiles no difference.  (Where more
// wavefronts have an item, halving them costs the second fetch of the positional terms: 2-3 % of a layer, read when heads followed one another.)
__device__ __forceinline__ bool split_items(int items, bool large_set, int waves) { return !large_set && 2 * items <= waves; }
// The attention phase's items -- (set, query tile, group of heads) -- are numbered set by set.  A set's table word: first row
// (bits 0-7), distinct voxels (8-15) and the number of its first item (from 16 on); words past the last set hold
// kNoItem, above every item number.  A wavefront holds the table a word per lane and finds the set of an item by counting
// the sets that start at or before it.
constexpr unsigned kNoItem = 0x7fffu << 16;
__device__ __forceinline__ unsigned set_word(int r0, int nu, int first_item) { return (unsigned)r0 | (unsigned)nu << 8 | (unsigned)first_item << 16; }
constexpr int kComputeUnits = 256;               // MI355X
constexpr int kLayerWaves = 12;                  // three per SIMD: one workgroup per CU (LDS), the other wavefronts hide one's waits

// erf-GELU (appendix "Network Architecture": the MLP of a DSVT layer) for bf16 features by linear
// interpolation: kGeluKnots intervals of width 1 / kGeluScale over [-4, 4), each with the slope
// and intercept of the chord through the exact values at its ends; below -4 + 1/64 the result is 0, from
// 4 - 1/64 on it is x - 6.5e-7 (both within 1.35e-4 of the exact function, from which x itself is 1.353e-4 away at the interval's
// lower end and x - 6.5e-7 is 1.347e-4; the chords are within 3.5e-5).  The
// table (4 KB) sits in LDS during the MLP: a lookup and one fma replace a dozen ALU instructions.
constexpr int kGeluKnots = 512;
constexpr float kGeluScale = 64.f;
__global__ void k_pack_gelu_table(float2* __restrict__ tab) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kGeluKnots) return;
  const double x0 = (i - kGeluKnots / 2 - 0.0625) / (double)kGeluScale, x1 = x0 + 1.0 / kGeluScale;   // (see gelu_entry)
  const double g0 = 0.5 * x0 * (1.0 + erf(x0 * 0.70710678118654752440)), g1 = 0.5 * x1 * (1.0 + erf(x1 * 0.70710678118654752440));
  const double sl = (g1 - g0) * kGeluScale;
  float2 e = make_float2((float)sl, (float)(g0 - sl * x0));
  if (i == 0) e = make_float2(0.f, 0.f);                      // x < -4 + 1/64 (and everything below)
  if (i == kGeluKnots - 1) e = make_float2(1.f, -6.5e-7f);    // x >= 4 - 1/64 (and everything above)
  tab[i] = e;
}
// The table's LDS address out of a float's mantissa: with 2^23 + address added, 8 * kGeluScale * x lands there in whole bytes, and an
// AND leaves the entry's address.  (The sum is rounded to the nearest byte, so intervals begin half a byte of x, 1/1024, below
// the multiples of 1/64, and the table's knots lie there.  Largest error over all x 1.347e-4, in the tails, root mean square over
// N(0, 1.2^2) 1.105e-5, both as with truncation to the index.)  Four instructions and a lookup; truncating to an index took five.  Pass
// of the 30,000-pillar frame 365.9 -> 363.6 us, 120,000 voxels 660.5 -> 655.1, skewed batch 7,380 -> 7,334.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(3))) f32x2* lds_pair;
typedef const __attribute__((address_space(3))) unsigned char* lds_byte;
__device__ __forceinline__ float gelu_start(const unsigned char* tab) {        // of every lookup: 2^23 + address of the interval of x = 0
  const unsigned at = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)tab;
  return __uint_as_float(0x4B000000u + at + kGeluKnots / 2 * 8);
}
__device__ __forceinline__ f32x2 gelu_entry(float start, float x) {          // the result is entry.x * x + entry.y
  constexpr float kEnd = kGeluKnots / 2 / kGeluScale;
  const float t = fmaf(__builtin_amdgcn_fmed3f(x, -kEnd, kEnd - 0.125f / kGeluScale), 8.f * kGeluScale, start);
  return *(lds_pair)(uintptr_t)(__float_as_uint(t) & 0x3FFF8u);
}

// The tiles of a workgroup of a full grid (kComputeUnits or twice as many workgroups; tiles are listed most rows first).  Its first tile is the one of its
// number.  Of the others n_tiles % grid workgroups, those with the smallest first tiles, take one more than the rest, and theirs are
// n_more consecutive ones from `first` on (counted behind the first tiles); the rest take what lies before and behind.  Both go back and forth, every
// second of their rounds in reverse, and `first` is chosen so that the two kinds of workgroups end together (first_of_more()).  Whatever
// `first` is, every tile is taken once.
struct Shares {
  int rounds, more, n_more;                  // whole rounds, workgroups with a tile more, how many tiles those take behind their first ones
  int grid;
  __device__ __forceinline__ Shares(int n_tiles, int grid_) : rounds(n_tiles / grid_), more(n_tiles % grid_), n_more(rounds * more), grid(grid_) {}
  __device__ __forceinline__ int others() const { return (rounds - 1) * (grid - more); }           // tiles behind the first ones that the rest take
  // tile number `round` >= 1 of workgroup b, -1: there is none
  __device__ __forceinline__ int tile(int b, int round, int first) const {
    const bool has_more = b >= grid - more;
    const int width = has_more ? more : grid - more, at = has_more ? b - (grid - more) : b, t = round - 1;
    if (t >= (has_more ? rounds : rounds - 1)) return -1;
    const int j = t * width + ((t & 1) != 0 ? at : width - 1 - at);
    return grid + (has_more ? first + j : (j < first ? j : j + n_more));
  }
};
// A wavefront chooses `first` from the rows of 64 tiles spread evenly over the list (rows: of tile (2 lane + 1) n_tiles / 128): the cost of a run of
// tiles from their prefix sums, a tile costing its rows and what 31 rows do (11.5 k clocks beside 372 a row at C = 192), for 64 places of the run.
// The rounds' sums differ by the last, partial round otherwise: of 6.26 rounds of the 120,000-voxel frame the slowest workgroup took 290 k clocks,
// the mean 263 k.  Back and forth through the list -> this: passes of 120,000 voxels 641.6 -> 622.3 us, four frames 1,044 -> 1,008, skewed batch 7,005 -> 6,939.
__device__ __forceinline__ int first_of_more(const Shares& sh, int n_tiles, int rows) {
  const int lane = threadIdx.x & 63;
  const float cost = (float)(rows < 0 ? 0 : (rows > kRowsMax ? kRowsMax : rows)) + 31.f, per = (float)n_tiles * (1.f / 64.f);
  float before = cost;                             // inclusive sums over the lanes
#pragma unroll
  for (int d = 1; d < 64; d *= 2) {
    const float t = __shfl_up(before, d, 64);
    if (lane >= d) before += t;
  }
  before -= cost;
  const auto prefix = [&](int k) {                 // cost of the first k tiles
    const float y = (float)k / per;
    int i = (int)y;
    i = i > 63 ? 63 : i;
    return (__shfl(before, i, 64) + (y - (float)i) * __shfl(cost, i, 64)) * per;
  };
  const int first = lane * sh.others() / 63;
  const float more = (prefix(sh.grid) - prefix(sh.grid - sh.more) + prefix(sh.grid + first + sh.n_more) - prefix(sh.grid + first));
  const float rest = prefix(n_tiles) - more;
  float worst = fmaxf(more / (float)sh.more, rest / (float)(sh.grid - sh.more));
  int best = first;
#pragma unroll
  for (int d = 1; d < 64; d *= 2) {                // the smallest, of equal ones the first
    const float w = __shfl_xor(worst, d, 64);
    const int f = __shfl_xor(best, d, 64);
    if (w < worst || (w == worst && f < best)) { worst = w; best = f; }
  }
  return best;
}

// Inclusive sum over the first 32 lanes of a wavefront (data-parallel-primitive shifts inside rows of 16 lanes, then lane 15's into
// the second row).
__device__ __forceinline__ int half_wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0x2, 0xF, false);
  return v;
}

struct LayerDev {
  const void *w_qkv, *w_o, *w_1, *w_2;       // packed (see mma.h)
  const float *b_qkv, *b_o, *b_1, *b_2, *ln1_g, *ln1_b, *ln2_g, *ln2_b, *rel_bias;
  const float2* gelu_tab;                    // kGeluKnots (slope, intercept) pairs, see k_pack_gelu_table
  float ln_eps;
  // position table [heads / 4][index][4], an index in bytes of a row of four heads (below 2^32): index of (q, k) = code(q) - code(k) + rel_const, at most
  // rel_last; rel_none: the row of -inf, the last one
  unsigned rel_const, rel_last, rel_none;
  int rel_my, rel_mz;
};

struct PositionTable { const float* rel_bias; unsigned rel_const, rel_last, rel_none; };     // what attention takes of LayerDev

struct MapsDev {
  const int32_t *set_inds, *n_sets, *n_tiles, *tile_desc;
  int32_t max_sets, max_tiles, tau, n_voxels;
};

template <typename T> struct LayerCall {
  LayerDev layer;
  MapsDev maps;
  const int4* coords;
  const T* x;
  T* out;                                    // may be x: a tile's rows are read, then written, by one workgroup only, and the tiles share no rows
  int full_layer;
};
// The kernel's one argument where it lies in memory.  Behind an empty asm, so that inside the loop over tiles a pointer is loaded where it is
// used: the compiler otherwise loads all of them in front of the loop and spills what the scalar registers do not hold into lanes of vector
// registers, 18 to 30 of them a kernel and two vector instructions each time one is needed.  With -> without: 3,001 pillars 151.1 ->
// 147.2 us, pillar frame 355.0 -> 351.1, hybrid windows 496.7 -> 488.7, four frames 1,079 -> 1,069, voxel frame 659.8 -> 648.4, skewed batch
// 7,616 -> 7,508, one block of 2,000 voxels in fp32 48.9 -> 47.9; attention of 4,000 voxels without a work list, C = 64, 10.1 -> 9.7.
template <typename T> __device__ __forceinline__ const __attribute__((address_space(4))) LayerCall<T>* layer_call() {
  auto call = (const __attribute__((address_space(4))) LayerCall<T>*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(call));
  return call;
}

template <typename T, int C, int HEADS, int HID> struct LayerLds {
  static constexpr int D = C / HEADS;
  static constexpr int PAD = lds_pad<T>();
  static constexpr int LDX = C + PAD;            // pitch of [row][feature] tiles, elements of T
  static constexpr int LDV = kRowsMax + 16 / (int)sizeof(T);   // pitch of V^T [feature][row]
  static constexpr int LDH = HID + PAD;          // pitch of the MLP hidden tile
  static constexpr size_t kTile = (size_t)kRowsMax * LDX * sizeof(T);
  // X and Q change places from one tile of a workgroup to the next (K stays between them): the rows of the next tile are
  // stored over this one's Q, and the MLP's hidden tile covers K and Q whichever side Q is on.
  static constexpr size_t off_k = kTile, off_v = 3 * kTile;
  static constexpr size_t kVt = (size_t)C * LDV * sizeof(T);
  static constexpr size_t off_misc = off_v + kVt;
  static constexpr size_t kRowTab = (size_t)(3 * kRowsPad + kHdrWords) * 4;       // rows' voxels, position codes, counts; header
  // of this tile and of the next one; 16 zero bytes, a place for results nobody needs (see attn_item), set table
  static constexpr size_t off_zero = off_misc + 2 * kRowTab, off_spare = off_zero + 16, kSpare = (size_t)C / 2 * sizeof(T) + 16 * sizeof(T);
  static constexpr size_t off_sets = off_spare + kSpare, kMisc = off_sets + (size_t)(kSetWords + 4) * 4 - off_misc;
  // after attention the V^T region holds the GELU table, the two LayerNorms' scales and shifts, and the LayerNorm statistics
  static constexpr size_t off_gelu = off_v, off_aff = off_v + 4096, off_stat = off_aff + (size_t)4 * C * 4, kStat = (size_t)2 * kStatGroupsMax * kRowsMax * 4;
  static_assert(off_stat + kStat <= off_misc, "GELU table and LayerNorm statistics must fit in the V^T region");
  static constexpr size_t total = off_misc + kMisc;
  static_assert((size_t)kRowsMax * LDH * sizeof(T) <= 2 * kTile, "hidden tile must fit in Q + K");
  static_assert(C % 64 == 0 && D % Mma<T>::KL == 0 && D % 4 == 0, "shape");
  static_assert(total <= 160 * 1024, "LDS of one CU");            // C = 192: 163,328 bytes, 512 below it
};

// Whether a tile leaves room in the LDS for a second workgroup on the compute unit: C = 64 in bf16.
template <typename T, int C, int HEADS, int HID> constexpr bool two_groups_fit() { return 2 * LayerLds<T, C, HEADS, HID>::total <= 160 * 1024; }

// Key tiles of the largest set in a tile whose items may be split (split_items).  At C = 64 in bf16 an item of a quarter of the heads is a
// single head, and it is a workgroup beside it on the compute unit, not idle wavefronts, that fills its waits: sets of three key tiles
// stay whole there, and so does every set once there are two workgroups to a compute unit (n_tiles > 256).  All split -> so, replayed blocks of
// two layers: 3,000 voxels in 30 x 30 windows, sets of up to 48, 15.8 -> 15.3 us; 27,000 and 45,000 of them, and 60,000 in 12 x 12 windows, no difference any more (40.1 -> 36.2,
// 49.9 -> 42.7 and 49.5 -> 47.2 when heads followed one another); never split: 300 voxels 11.75 -> 11.7.  The other shapes, never split -> as here, 500 and 3,000 voxels spread evenly over 12 x 12
// windows: C = 192 20.4 -> 20.45 and 25.7 -> 25.6, C = 128 and fp32 within 0.1 (25.0 -> 24.4, 33.2 -> 32.3 and the like before).
template <typename T, int C, int HEADS, int HID> constexpr int split_key_tiles() { return two_groups_fit<T, C, HEADS, HID>() ? 2 : 3; }

// LDS by its 32-bit address: constants added to it become the instruction's offset.
template <typename V> __device__ __forceinline__ V lds_read(int at) { return *(const __attribute__((address_space(3))) V*)(uintptr_t)(unsigned)at; }
template <typename V> __device__ __forceinline__ void lds_write(int at, V v) { *(__attribute__((address_space(3))) V*)(uintptr_t)(unsigned)at = v; }

// Attention of one (set, query tile, group of heads) item (Eq. 5): for each of its heads,
// logits = Q K^T (+ PE), softmax over the set's distinct voxels, O = P V; O overwrites the Q
// entries it was computed from.  KTC = key tiles of the set (compile time: no branches inside).
// S^T is produced key-major (keys as MFMA rows) so that a lane holds 4 keys of ONE query: the
// softmax reductions are in-lane plus two cross-lane steps, and P^T is already laid out as the B
// operand of O^T = V^T P^T.  Q arrives scaled by log2(e) / sqrt(d) (the projection's epilogue does
// it), and the positional term -- which depends on (query, key) only through the coordinate
// difference -- comes from a table, one row of four heads per pair, fetched once for all heads of the item.  The keys past
// the set's last voxel take the table's extra last row, which holds -inf: no mask arithmetic.
// DUP: repeated slots count as keys (the exponentials are multiplied by the slots' counts).
// One basic block: lanes past the head width read their queries from 16 zero bytes, and queries that do not exist are written
// to a spare place, so that nothing stands between the heads and their instructions mix.  Everything a head adds to an
// address is a constant, i.e. an offset in the instruction.
// What bounds it is the issue of vector instructions (an item of two key tiles and four heads: 36 exp and rcp at a quarter of the rate and
// 250 others, 3 wavefronts a SIMD) and, within a head, one dependent step after the other.  So the heads go through the steps side by side -- all
// products with the keys, all maxima, .. --, the heads' maxima share the lane swaps (col_reduce()), the terms are added behind the
// products (as the MFMAs' start values they had to be moved into place, an instruction each too, and to be there first).  The sums are of the 32-bit
// probabilities, in one order of keys and lanes whatever the heads an item has (from the matrix cores, of those rounded to bf16: the same time in large sets, a value off by
// up to 2^-8).  Head after head, 336 + 36 instructions and 46 waits -> this,
// attention of a 64-row tile 7.6 -> 6.3 k clocks, of an 82-row tile 10.5 -> 9.0 k; passes of 3,001 pillars 141.9 -> 138.7 us, 30,000 337.6 -> 330.5,
// windows of 12 and 24 cells 472.8 -> 458.1, 30 x 30 windows 267.7 -> 265.0, 120,000 voxels 619.7 -> 604.1.  Position
// table rows of all heads -> of four: 30 x 30 windows 264.8 -> 261.2 (a table of 111 KB: the rows that a load touches lie in half as many
// lines), 12 x 12 windows no difference.
// Tried: the first item's positional terms requested in front of the output projection's weights, behind which they come back -- 48 more
// registers across the barrier, spills, and with those weights requested behind the attention instead no gain.
template <typename T, int C, int HEADS, int HID, int KTC, int HG, bool DUP>
__device__ __forceinline__ void attn_item(const PositionTable& p, unsigned char* smem, int q_off, const int32_t* row_code,
                                          const float* row_mult, int r0, int nu, int qt, int hh, int rows_ready) {
  typedef LayerLds<T, C, HEADS, HID> L;
  typedef Mma<T> M;
  typedef typename M::Frag Frag;
  typedef typename M::Vec4 Vec4;
  constexpr int D = L::D, KC = M::KC, KL = M::KL, ES = (int)sizeof(T);
  constexpr int PX = L::LDX * ES, PV = L::LDV * ES;                // row pitches in bytes
  constexpr int TPC = KC / 16;                    // key tiles per PV fragment: 2 (bf16) or 1 (fp32)
  static_assert(HG == 1 || HG == 2 || HG == 4, "heads per item");
  static_assert(D <= KC, "one fragment per query");
  // Four heads of four key tiles and more take the keys 32 at a time, with a running maximum: all logits at once do not fit the registers
  // (and two heads at a time fetch the terms twice as often, 8 bytes a lane; a load is 17 clocks of the compute unit's memory pipe either way).
  constexpr int CT = HG == 4 && KTC > 3 ? 2 : KTC;                // key tiles at a time
  constexpr int HS = C == 192 && KTC > 4 ? 1 : HG;                // heads side by side (two of five or six key tiles, C = 192: no difference, 84.6 us a block either way)
  static_assert(CT == KTC || HS == HG, "a running maximum per head");
  const int lane = opaque_tid() & 63, m = lane & 15, g = lane >> 4;
  const int qi = 16 * qt + m;
  const int qrow = r0 + (qi < nu ? qi : nu - 1);
  const int h0 = hh * HG * D * ES;                // this item's heads in a row

  // The keys' positional terms, one table row per (query, key) for all heads of the item
  typedef float Terms __attribute__((ext_vector_type(HG)));          // (indexed by head)
  const unsigned qc = (unsigned)row_code[qrow] + p.rel_const;
  const int left = nu - (16 * (KTC - 1) + 4 * g);                  // keys of the last tile from this lane's first on
  const char* tab = reinterpret_cast<const char*>(p.rel_bias) + (size_t)(hh * HG / 4) * ((size_t)p.rel_none + kRelRow) + hh * HG % 4 * 4;
  Terms bias[CT][4];
  const auto fetch_terms = [&](int k0) {
#pragma unroll
    for (int kt = k0; kt < k0 + CT && kt < KTC; ++kt) {
      const int4 kl = *reinterpret_cast<const int4*>(row_code + r0 + 16 * kt + 4 * g);
      const int kls[4] = {kl.x, kl.y, kl.z, kl.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        unsigned at = min(qc - (unsigned)kls[i], p.rel_last);      // (modulo 2^32: right for every index of the table)
        if (kt == KTC - 1) at = i < left ? at : p.rel_none;        // only the last key tile is ragged
        bias[kt - k0][i] = *reinterpret_cast<const Terms*>(tab + at);
      }
    }
  };
  fetch_terms(0);
  const int lds0 = (int)(uintptr_t)(lds_byte)smem;
  const bool live = g * KL < D;                   // lanes past the head width
  // Addresses in swizzled rows, of the item's first head and (a head is an odd number of 16-byte pieces) of its second one: every other head on is
  // a constant away.
  constexpr int HB = D * ES, PAR = HB % 32 != 0 ? 2 : 1;
  static_assert(L::off_k % 32 == 0 && PX % 32 == 0, "addresses are swizzled like places in a row");
  const auto swizzled = [](int at, int row) { return at ^ (row & 4) << 2; };
  int q_at[PAR], k_first[PAR], k_last[PAR];
  const int k_row = r0 + min(16 * (KTC - 1) + m, nu - 1);
#pragma unroll
  for (int par = 0; par < PAR; ++par) {
    const int piece = lds0 + h0 + par * HB + (live ? g * KL * ES : 0);       // (dead k lanes: finite K times the zero Q)
    q_at[par] = live ? swizzled(q_off + qrow * PX + piece, qrow) : lds0 + (int)L::off_zero;
    k_first[par] = swizzled((int)L::off_k + (r0 + m) * PX + piece, r0 + m);
    k_last[par] = swizzled((int)L::off_k + k_row * PX + piece, k_row);
  }
  const int q_step = live ? PAR * HB : 0;
  const auto k_at = [&](int h, int kt) { return (kt < KTC - 1 ? k_first[h % PAR] + 16 * kt * PX : k_last[h % PAR]) + h / PAR * PAR * HB; };
  // Key columns past the tile's rows hold no V: their P is an exact zero, so any finite column will do, and the set's first
  // one is read instead.  (Rows past the head width: the tile's row of a lane below it; results thrown away.)
  constexpr int DT = (D + 15) / 16;
  int v_first[DT], v_last[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const int dv = 16 * dt + m, row = lds0 + (int)L::off_v + hh * HG * D * PV + (dv < D ? dv : m) * PV + r0 * ES;
    v_first[dt] = row + 4 * g * ES;
    v_last[dt] = row + (r0 + 16 * (KTC - 1) + 4 * g < rows_ready ? 16 * (KTC - 1) + 4 * g : 0) * ES;
  }
  const auto v_at = [&](int dt, int kt) { return kt < KTC - 1 ? v_first[dt] + 16 * kt * ES : v_last[dt]; };
  int o_at[DT][PAR];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int par = 0; par < PAR; ++par)
      o_at[dt][par] = qi < nu && 16 * dt + 4 * g < D ? swizzled(lds0 + q_off + qrow * PX + h0 + par * HB + (16 * dt + 4 * g) * ES, qrow) : lds0 + (int)L::off_spare + par * HB;

#pragma unroll
  for (int hb = 0; hb < HG; hb += HS) {
    constexpr f32x4 kZero = {0.f, 0.f, 0.f, 0.f};
    float mx[HS], sum[HS];                          // of the keys so far
    f32x4 O[HS][DT];                                // O^T[dv][q] = sum_key V^T[dv][key] P^T[key][q]
#pragma unroll
    for (int k0 = 0; k0 < KTC; k0 += CT) {
      constexpr int NCH = (CT + TPC - 1) / TPC;     // PV fragments
      const int kn = KTC - k0 < CT ? KTC - k0 : CT;
      f32x4 S[HS][CT];                              // S[hl][kt][i]: key 16*(k0 + kt) + 4*g + i, query 16*qt + m
#pragma unroll
      for (int hl = 0; hl < HS; ++hl) {
        const Frag fq = lds_read<Frag>(q_at[(hb + hl) % PAR] + (hb + hl) / PAR * q_step);
#pragma unroll
        for (int kt = 0; kt < kn; ++kt) S[hl][kt] = M::mma(lds_read<Frag>(k_at(hb + hl, k0 + kt)), fq, kZero);
      }
      // S + terms: the logits in units of log2(e), -inf for the keys that do not exist: exp is a bare exp2
      float cm[HS];
#pragma unroll
      for (int hl = 0; hl < HS; ++hl) {
#pragma unroll
        for (int k = 0; k < 4 * kn; ++k) {
          const float x = S[hl][k >> 2][k & 3] + bias[k >> 2][k & 3][hb + hl];
          S[hl][k >> 2][k & 3] = x;
          cm[hl] = k == 0 ? x : fmaxf(cm[hl], x);
        }
      }
      // (Key 0 exists for every query, but the table may hold -inf for it and for all keys of a step.  The running maximum is kept at the lowest float or
      // above, which no finite logit lies below: -inf less it stays -inf, where -inf less -inf is NaN, and nothing of such a step counts in the next one.)
      col_reduce(cm, [](float a, float b) { return raw_max(a, b); }, [](float a) { return CT < KTC ? raw_max(a, -FLT_MAX) : a; });
      float scale[HS];                              // of the keys before these
#pragma unroll
      for (int hl = 0; hl < HS; ++hl) {
        if (k0 > 0) {
          cm[hl] = raw_max(cm[hl], mx[hl]);
          scale[hl] = __builtin_amdgcn_exp2f(mx[hl] - cm[hl]);
          sum[hl] *= scale[hl];
        }
        mx[hl] = cm[hl];
      }
      Frag fp[HS][NCH];
#pragma unroll
      for (int hl = 0; hl < HS; ++hl) {
#pragma unroll
        for (int kt = 0; kt < kn; ++kt) {
          f32x4 mult;
          if constexpr (DUP) mult = *reinterpret_cast<const f32x4*>(row_mult + r0 + 16 * (k0 + kt) + 4 * g);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float e = __builtin_amdgcn_exp2f(S[hl][kt][i] - mx[hl]);       // exp2(-inf) = 0
            S[hl][kt][i] = DUP ? e * mult[i] : e;
            // (the fma written out: left to itself the compiler makes one of either product of the first two, and not the same one in every kernel)
            sum[hl] = k0 + kt + i == 0 ? S[hl][kt][i] : (DUP ? __builtin_fmaf(e, mult[i], sum[hl]) : sum[hl] + e);
          }
          // (The sum up to here stands before the next key tile's: the compiler otherwise adds behind all conversions and keeps the 32-bit probabilities until
          // then, and C = 128 spills 37 registers, 73 with repeats as keys, C = 64 in kSets96Slim four.)
          if (KTC > 3) asm volatile("" : "+v"(sum[hl]));
        }
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          if constexpr (TPC == 2) {
            const f32x4 p0 = S[hl][2 * c < kn ? 2 * c : 0], p1 = 2 * c + 1 < kn ? S[hl][2 * c + 1 < kn ? 2 * c + 1 : 0] : kZero;
            fp[hl][c] = Frag{(bf16_t)p0[0], (bf16_t)p0[1], (bf16_t)p0[2], (bf16_t)p0[3], (bf16_t)p1[0], (bf16_t)p1[1], (bf16_t)p1[2], (bf16_t)p1[3]};
          } else {
            fp[hl][c] = S[hl][c];
          }
        }
      }
      if (k0 + CT < KTC) fetch_terms(k0 + CT);
#pragma unroll
      for (int hl = 0; hl < HS; ++hl) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          f32x4 o = k0 > 0 ? O[hl][dt] * scale[hl] : kZero;
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            if (c * TPC >= kn) continue;
            Frag fv;
            if constexpr (TPC == 2) {
              const bf16x4 lo = lds_read<bf16x4>(v_at(dt, k0 + 2 * c) + (hb + hl) * D * PV);
              bf16x4 hi = {0, 0, 0, 0};
              if (2 * c + 1 < kn) hi = lds_read<bf16x4>(v_at(dt, k0 + 2 * c + 1) + (hb + hl) * D * PV);
              fv = Frag{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            } else {
              fv = lds_read<Frag>(v_at(dt, k0 + c) + (hb + hl) * D * PV);
            }
            o = M::mma(fv, fp[hl][c], o);
          }
          O[hl][dt] = o;
        }
      }
      if (CT < KTC) __builtin_amdgcn_sched_barrier(0);             // (156 registers, 160 with repeats as keys; without it a few more, a block 58.5 us either way)
    }
    col_reduce(sum, [](float a, float b) { return a + b; }, [](float a) { return __builtin_amdgcn_rcpf(a); });
#pragma unroll
    for (int hl = 0; hl < HS; ++hl)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) lds_write<Vec4>(o_at[dt][(hb + hl) % PAR] + (hb + hl) / PAR * PAR * HB, pack4<T>(O[hl][dt] * sum[hl]));
  }
}

// An item of a set with kts key tiles: up to three key tiles half of the heads per item (split_items: a quarter), beyond that
// big_heads().
template <typename T, int C, int HEADS, int HID, SetSize SETS, bool DUP>
__device__ __forceinline__ void attn_any(const PositionTable& p, unsigned char* smem, int q_off, const int32_t* row_code,
                                         const float* row_mult, int r0, int nu, int qt, int hh, int kts, bool split, int rows_ready) {
  constexpr int HG2 = HEADS / 2, HG4 = HEADS / 4, HGB = big_heads(C, DUP, SETS);
  if (split) {
    if (kts == 1) attn_item<T, C, HEADS, HID, 1, HG4, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
    else if (kts == 2) attn_item<T, C, HEADS, HID, 2, HG4, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
    else attn_item<T, C, HEADS, HID, 3, HG4, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
  } else if (kts == 1) attn_item<T, C, HEADS, HID, 1, HG2, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
  else if (kts == 2) attn_item<T, C, HEADS, HID, 2, HG2, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
  else if (SETS == kSets48 || kts == 3) attn_item<T, C, HEADS, HID, 3, HG2, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
  else if constexpr (SETS != kSets48) {
    if (kts == 4) attn_item<T, C, HEADS, HID, 4, HGB, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
    else if (kts == 5) attn_item<T, C, HEADS, HID, 5, HGB, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
    else attn_item<T, C, HEADS, HID, 6, HGB, DUP>(p, smem, q_off, row_code, row_mult, r0, nu, qt, hh, rows_ready);
  }
}

// Workgroups that share a compute unit, by LDS and registers: with two, each may use 80 registers a thread.
template <typename T, int C, int HEADS, int HID> constexpr int groups_per_cu(SetSize sets) {
  return sets != kSets96 && two_groups_fit<T, C, HEADS, HID>() ? 2 : 1;
}

// SETS: the instantiations for sets of four to six key tiles; the common one does not carry that code.
//
// The grid is as many workgroups as fit the GPU at once; each takes every gridDim.x-th tile, back and forth (tiles are listed
// most rows first), LONG: the tiles Shares says.  What bounds it is not one unit but the chain of a tile's phases; a tile's beginning -- descriptor, then the
// rows it names, then weights -- takes 8 k of the 42 k clocks of a workgroup's only 64-row tile, and between two tiles of a workgroup all of it is
// under way during the tile before: the descriptor is requested behind the attention, the rows behind the first MLP matrix
// (stored over Q once the second one is through with it; X and Q change places), the Q/K/V weights around the last LayerNorm.
// The rows of a tile leave from registers, 16 bytes a lane, so no tile waits for a copy through LDS.  One tile a workgroup
// -> this loop, pass of the 30,000-pillar frame (two tiles a workgroup) 360.0 -> 359.1 us, four frames 1,109 -> 1,078, 30 x 30
// windows 316.9 -> 290.0, 120,000 voxels 679 -> 653, skewed batch 7,686 -> 7,383; 3,001 pillars (one tile a workgroup)
// 158.5 -> 160.1, of which the kernel's own time is 16.0 -> 15.9 a layer.
// LONG: the frame has two full rounds of tiles and more (is_long()).
template <typename T, int C, int HEADS, int HID, int NT_QKV, int NT_O, int NT_1, int NT_2, SetSize SETS, bool DUP, bool LONG>
__device__ __forceinline__ void layer_tiles(const LayerCall<T>& call) {
  const LayerDev& p = call.layer;
  const MapsDev& mp = call.maps;
  typedef LayerLds<T, C, HEADS, HID> L;
  typedef typename Mma<T>::Vec4 Vec4;
  constexpr int LDX = L::LDX, LDV = L::LDV, LDH = L::LDH;
  constexpr int NW = kLayerWaves, NTHREADS = NW * 64;
  // LayerNorm phases: SG feature groups x RS parts of the row tiles (C = 192 six groups and halves, else four and thirds), one
  // item per wavefront.  (Halves leave a third of the wavefronts of C <= 128 without an item: C = 128, 46,827 pillars
  // 399.2 -> 384.7 us, 11,491 pillars 155.6 -> 151.1, 30 x 30 windows 282.0 -> 280.8.  The first MLP matrix in the same parts, each
  // fragment then loaded three times: 395.0, 154.0 and 286.1: it keeps all rows per wavefront.)
  constexpr int SG = C / (16 * NT_O), RS = NW / SG, kOwnTiles = kRowTiles / RS;
  static_assert(NT_O == NT_2 && SG * 16 * NT_O == C && RS * SG == NW && RS * kOwnTiles == kRowTiles && SG <= kStatGroupsMax, "LayerNorm phases: one item per wavefront");
  extern __shared__ __align__(32) unsigned char smem[];             // (addresses are swizzled like places in a row)
  T* Ks = reinterpret_cast<T*>(smem + L::off_k);
  T* Vt = reinterpret_cast<T*>(smem + L::off_v);
  float* stat = reinterpret_cast<float*>(smem + L::off_stat);           // over V^T once attention is done
  unsigned* set_tab = reinterpret_cast<unsigned*>(smem + L::off_sets);   // [kSetWords + 4]: set_word() of every set, number of items, whether they are split; LONG: the next tile, Shares' `first`

  // wave-uniform values are read back through readfirstlane so that the compiler keeps them in
  // scalar registers: branches on them are scalar branches, not exec-mask divergence
  int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#define DSVT_REFRESH_LANE() do { tid = opaque_tid(); lane = tid & 63; m = lane & 15; g = lane >> 4; } while (0)
  typedef GemmPhase<T, NT_QKV, C, 3 * C, NW, 1, 1, true> QkvPhase;
  // The first two output tiles of every wavefront's Q/K/V weights (C = 192: of three, C = 128: both, C = 64: the only one)
  // of a workgroup's first tile are requested behind the descriptor, and arrive during the two dependent trips to memory (descriptor, then the rows it
  // names) in which the compute unit's memory pipeline would have nothing else to do: it takes a 1 KB fragment every ~19
  // cycles, 2.7 k cycles for the 144 of C = 192, about what the descriptor needs to come back.  C = 192, pass of the
  // 30,000-pillar frame / of the 120,000-voxel one, a tile a workgroup: none ahead 378.5 / 732 us, one tile 370.0 / 720, two 368.6 / 712, all
  // three 372.2 / 717 (the rows' requests queue behind them).  C = 128 (96 fragments in all), a block of the 30,000-pillar
  // frame / of 20,000 voxels in 30 x 30 windows: none 61.2 / 67.3 us, one tile 60.4 / 66.7, both 59.9 / 65.7.  C = 64, a block of
  // 30,000 pillars: bf16 28.1 us without, 28.2 with, 2,000 pillars 16.1 and 15.9; fp32 78.9 and 78.0.
  constexpr int kEarly = NT_QKV < 2 ? NT_QKV : 2;

  // The arguments (four cache lines) in one go, then the number of tiles and the first tile's descriptor together: three waits less in a
  // row.  Passes: pillar frame 348.8 -> 347.8 us, hybrid windows 490.1 -> 488.2, 4,137 pillars 74.4 -> 73.6.
  int tile = blockIdx.x;
  asm("" : "+s"(tile) : "s"(p.w_qkv), "s"(p.gelu_tab), "s"(mp.tile_desc), "s"(mp.n_tiles), "s"(mp.max_tiles), "s"(mp.tau), "s"(call.x));
  const bool listed = mp.tile_desc != nullptr;
  const int per_wg = fixed_sets(mp.tau);         // without a work list a tile is two sets
  int n_tiles, n_sets = 0, word = 0;
  if (listed) {
    n_tiles = *mp.n_tiles;
    if (tid < 256) word = mp.tile_desc[(size_t)tile * 256 + tid];
    n_tiles = n_tiles < mp.max_tiles ? n_tiles : mp.max_tiles;
  } else {
    n_sets = *mp.n_sets;
    n_sets = n_sets < mp.max_sets ? n_sets : mp.max_sets;
    n_tiles = (n_sets + per_wg - 1) / per_wg;
  }
  constexpr int kGrid = kComputeUnits * groups_per_cu<T, C, HEADS, HID>(SETS);       // workgroups, if there are more tiles than that
  int stride = LONG ? 1 : 2 * (int)(gridDim.x - blockIdx.x) - 1;      // to the next tile; LONG: the workgroup's tile number
  int xo = 0, tab = 0;                           // byte offsets of X (Q: the other side of K) and of this tile's row tables
  DSVT_PHASE(tile, 0);

  // the row tables of a tile from its descriptor, a word per thread of the first four wavefronts
  const auto row_vox = [&](int t) { return reinterpret_cast<int32_t*>(smem + L::off_misc + t); };
  const auto row_code = [&](int t) { return row_vox(t) + kRowsPad; };
  const auto row_mult = [&](int t) { return reinterpret_cast<float*>(row_vox(t) + 2 * kRowsPad); };
  const auto header = [&](int t) { return row_vox(t) + 3 * kRowsPad; };
  const auto store_desc = [&](int word, int t, int n_voxels) {
    if (tid < kHdrWords) {
      header(t)[tid] = word;
    } else if (tid < kHdrWords + 2 * kRowsMax) {     // words 64 + 2 r and 65 + 2 r: voxel and (slots << 24 | position code) of row r
      const int r = (tid - kHdrWords) >> 1;
      if ((tid & 1) == 0) {
        row_vox(t)[r] = (word >= 0 && word < n_voxels) ? word : -1;
      } else {
        row_code(t)[r] = (word & 0xFFFFFF) * kRelRow;
        if constexpr (DUP) row_mult(t)[r] = (float)((unsigned)word >> 24);
      }
    }
  };
  // rows and row tiles of a tile (no sets: no rows, and one row tile of zeros)
  const auto tile_rows = [&](int t) {
    const int ns = __builtin_amdgcn_readfirstlane(header(t)[1]), R = __builtin_amdgcn_readfirstlane(header(t)[0]);
    return ns <= 0 || R < 0 ? 0 : (R > kRowsMax ? kRowsMax : R);
  };
  const auto row_tiles = [](int R) { return R > 0 ? (R + 15) >> 4 : 1; };

  // gather (Eq. 4): rows of x -> LDS, 16 bytes per thread, dead rows zero.  The loads are unconditional (clamped addresses).
  // Thread t takes piece t % CH of the rows t / CH, t / CH + GR, ...
  constexpr int CH = C * (int)sizeof(T) / 16, GR = NTHREADS / CH, G = (kRowsMax + GR - 1) / GR;
  static_assert(NTHREADS % CH == 0 && kRowsMax % GR == 0, "whole rows per pass");
  const auto request_rows = [&](uint4 (&gv)[G], unsigned& live, int t, int RT, const T* x) {
    const int r0 = tid / CH, c = tid - r0 * CH;
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int v = r0 + k * GR < RT * 16 ? row_vox(t)[r0 + k * GR] : -1;
      live |= v >= 0 ? 1u << k : 0u;
      gv[k] = reinterpret_cast<const uint4*>(x + (size_t)(v >= 0 ? v : 0) * C)[c];
    }
  };
  const auto store_rows = [&](const uint4 (&gv)[G], unsigned live, int off, int RT) {
    static_assert(GR % 8 == 0, "a thread's rows are swizzled alike");
    const int r0 = tid / CH, c = (tid - r0 * CH) ^ (r0 >> 2 & 1);
#pragma unroll
    for (int k = 0; k < G; ++k)
      if (r0 + k * GR < RT * 16)
        *reinterpret_cast<uint4*>(smem + off + (r0 + k * GR) * LDX * (int)sizeof(T) + c * 16) = (live >> k & 1u) != 0u ? gv[k] : make_uint4(0u, 0u, 0u, 0u);
  };
  // A row of a tile from registers in accumulator layout -> the voxel's row of out; bf16 in 16-byte pieces: neighbouring 16-lane
  // rows exchange halves, so that a lane holds 8 consecutive features.  Two output tiles: of the first one in the even rows, of the
  // second in the odd ones.
  const auto put_out = [&](T* out, int t, int R, int row, int o0, const f32x4 (&v)[NT_O]) {
    const int vox = row < R ? row_vox(t)[row] : -1;
    if constexpr (NT_O == 2 && sizeof(T) == 2) {
      union { Vec4 h; unsigned u[2]; } a, b;
      a.h = pack4<T>(v[0]);
      b.h = pack4<T>(v[1]);
      const auto s0 = __builtin_amdgcn_permlane16_swap(a.u[0], b.u[0], false, false), s1 = __builtin_amdgcn_permlane16_swap(a.u[1], b.u[1], false, false);
      if (vox >= 0) *reinterpret_cast<uint4*>(out + (size_t)vox * C + o0 + 16 * (g & 1) + 8 * (g >> 1)) = make_uint4(s0[0], s1[0], s0[1], s1[1]);
    } else {
#pragma unroll
      for (int nt = 0; nt < NT_O; ++nt)
        if (vox >= 0) *reinterpret_cast<Vec4*>(out + (size_t)vox * C + o0 + 16 * nt + 4 * g) = pack4<T>(v[nt]);
    }
  };
  // One output tile (C = 64): row of one row tile in the even 16-lane rows and, if there is a next one, row + 16 of it in the odd ones.
  // 8 bytes a lane -> this: two layers of 100,000 voxels in 12 x 12 windows 70.8 -> 69.0 us, of 20,000 in 30 x 30 windows, sets of up to 48,
  // 27.0 -> 26.3; attention without a work list, 60,000 voxels, 20.7 -> 19.9 (a copy through LDS 20.1, and slower than 8 bytes in small frames).
  constexpr bool kPairs = NT_O == 1 && sizeof(T) == 2;
  static_assert(!kPairs || kOwnTiles == 2, "the row tiles of a wavefront are one pair");
  const auto put_pair = [&](T* out, int t, int R, int row, bool two, int o0, Vec4 v0, Vec4 v1) {
    union { Vec4 h; unsigned u[2]; } a, b;
    a.h = v0;
    b.h = v1;
    const int mine = row + 16 * (g & 1), vox = (two || (g & 1) == 0) && mine < R ? row_vox(t)[mine] : -1;
    const auto s0 = __builtin_amdgcn_permlane16_swap(a.u[0], b.u[0], false, false), s1 = __builtin_amdgcn_permlane16_swap(a.u[1], b.u[1], false, false);
    if (vox >= 0) *reinterpret_cast<uint4*>(out + (size_t)vox * C + o0 + 8 * (g >> 1)) = make_uint4(s0[0], s1[0], s0[1], s1[1]);
  };

  // ---- 3. Q, K, V = X W^T + b; V stored transposed
  const auto project = [&](QkvPhase& qkv, int RT) {
    const T* Xs = reinterpret_cast<const T*>(smem + xo);
    T* Qs = reinterpret_cast<T*>(smem + (2 * L::kTile - xo));
    // the V items run with exchanged MFMA operands: a lane then holds four consecutive rows of one
    // feature, i.e. 8 contiguous bytes of V^T (a plain store instead of four 2-byte ones)
    static_assert((C / 16) % NT_QKV == 0, "an item never straddles the Q/K/V boundary");
    const float q_scale = rsqrtf((float)L::D) * 1.4426950408889634f;
    const int o0 = wave * 16 * NT_QKV;
    // (part k of a row tile's epilogue takes output tile k - 1)
    const auto store = [&](T* dst, int r, int nt, const f32x4& v) { *reinterpret_cast<Vec4*>(dst + (16 * r + m) * LDX + 16 * nt + (4 * g ^ swizzle<T>(m))) = pack4<T>(v); };
    if (o0 >= 2 * C) {
      qkv.template run_rows<true, NT_QKV + 1>(Xs, LDX, RT, [&](int k, int r, f32x4 (&acc)[NT_QKV]) {
        if (k >= 1 && k <= NT_QKV) *reinterpret_cast<Vec4*>(Vt + (o0 - 2 * C + 16 * (k - 1) + m) * LDV + 16 * r + 4 * g) = pack4<T>(acc[k - 1]);
      });
    } else if (o0 >= C) {
      qkv.template run_rows<false, NT_QKV + 1>(Xs, LDX, RT, [&](int k, int r, f32x4 (&acc)[NT_QKV]) {
        if (k >= 1 && k <= NT_QKV) store(Ks + (o0 - C), r, k - 1, acc[k - 1]);
      });
    } else {
      qkv.template run_rows<false, NT_QKV + 1>(Xs, LDX, RT, [&](int k, int r, f32x4 (&acc)[NT_QKV]) {
        if (k >= 1 && k <= NT_QKV) store(Qs + o0, r, k - 1, acc[k - 1] * q_scale);      // logits in units of log2(e)
      });
    }
  };

  if (tile >= n_tiles) return;
  QkvPhase first(reinterpret_cast<const T*>(p.w_qkv), wave);
  first.template prefetch_first<kEarly>();
  if (tid < 4) reinterpret_cast<unsigned*>(smem + L::off_zero)[tid] = 0u;
  for (int r = kRowsMax + tid; r < kRowsPad; r += NTHREADS)
    for (int t = 0; t <= (int)L::kRowTab; t += (int)L::kRowTab) { row_vox(t)[r] = -1; row_code(t)[r] = 0; row_mult(t)[r] = 0.f; }

  if (listed) {
    // ---- 1a. rows from the tile descriptor the partition wrote for this tile (1 KB, one load)
    store_desc(word, tab, mp.n_voxels);
  } else {
    // ---- 1b. no work list: two sets per tile, rows derived from set_inds and coords
    // (A set's slots stay in its wavefront's registers.  Read a second time once the rows are numbered -> kept: C = 64 bf16, attention of 300 voxels
    // 5.44 -> 5.22 us, of 4,000 9.76 -> 9.34; C = 64 bf16, two layers of 20,000 voxels, sets of up to 64, 47.9 -> 46.6.)
    const int tau = mp.tau, s_begin = tile * per_wg, ns = n_sets - s_begin < per_wg ? n_sets - s_begin : per_wg;
    int32_t* hdr = header(tab);
    for (int r = tid; r < kRowsPad; r += NTHREADS) { row_vox(tab)[r] = -1; row_code(tab)[r] = 0; row_mult(tab)[r] = 0.f; }
    const int v = wave < ns && lane < tau ? mp.set_inds[(size_t)(s_begin + wave) * tau + lane] : -2;      // (a wavefront has one set at most)
    const int prev = __shfl_up(v, 1, 64);
    const bool first = wave < ns && lane < tau && (lane == 0 || v != prev), valid = first && v >= 0 && v < mp.n_voxels;   // repeats are adjacent
    const unsigned long long mask = __ballot(first);
    if (wave < ns && lane == 0) hdr[kHdrNu + wave] = __popcll(mask);
    lds_barrier();
    if (tid == 0) {
      int r = 0;
      for (int s = 0; s < ns; ++s) { hdr[kHdrR0 + s] = r; r += (hdr[kHdrNu + s] + 3) & ~3; }   // each set starts on a multiple of 4 rows
      hdr[0] = r;
      hdr[1] = ns;
    }
    lds_barrier();
    if (valid) {
      const int r = hdr[kHdrR0 + wave] + __popcll(mask & ((1ull << lane) - 1ull));
      const unsigned long long later = mask >> (lane + 1);
      const int run = later ? (__ffsll((long long)later)) : (tau - lane);   // slots holding this voxel
      const int4 c = call.coords[v];
      row_vox(tab)[r] = v;
      row_mult(tab)[r] = (float)run;
      row_code(tab)[r] = (int)((unsigned)((c.y * p.rel_my + c.z) * p.rel_mz + c.w) * (unsigned)kRelRow);
    }
  }
  lds_barrier();
  DSVT_PHASE(tile, 1);                             // rows known
  // ---- 2. gather
  int R = tile_rows(tab), RT = row_tiles(R);
  {
    uint4 gv[G];
    unsigned live = 0u;
    request_rows(gv, live, tab, RT, call.x);
    store_rows(gv, live, xo, RT);
  }
  lds_barrier();
  DSVT_REFRESH_LANE();
  DSVT_PHASE(tile, 2);                                 // rows in LDS
  first.template prefetch_rest<kEarly>(p.b_qkv, 2 * C / (16 * NT_QKV));
  if constexpr (LONG) {                            // (the second wavefront, which is early, finds out about the tiles)
    int sample;
    opaque_def(sample);
    const bool choose = wave == 1 && n_tiles > kGrid && n_tiles % kGrid != 0;
    if (choose) sample = mp.tile_desc[(size_t)((2 * lane + 1) * (int64_t)n_tiles / 128) * 256];
    project(first, RT);
    if (wave == 1) {
      int from = 0;
      if (choose) from = first_of_more(Shares(n_tiles, kGrid), n_tiles, sample);
      if (lane == 0) set_tab[kSetWords + 3] = (unsigned)from;      // (its own)
    }
  } else {
    project(first, RT);
  }

  for (;;) {
    DSVT_REFRESH_LANE();
    const auto args = layer_call<T>();
    const int full_layer = args->full_layer;
    T* Xs = reinterpret_cast<T*>(smem + xo);
    T* Qs = reinterpret_cast<T*>(smem + (2 * L::kTile - xo));
    T* Hs = reinterpret_cast<T*>(smem + (L::kTile - xo / 2));
    int next = LONG ? 0 : tile + stride;
    bool more = LONG || next < n_tiles;
    // LayerNorm phases (small weight matrices): every wavefront owns C / SG features of one part of
    // the row tiles; the Q/K/V and first MLP projections (bandwidth-heavy) give a wavefront all rows
    // of its output tiles instead, so that each of their weight fragments is loaded only once.  The last part may have fewer
    // row tiles than the others, or none: its wavefronts request no weights (C = 192, a tile of a single row tile: 220 KB of the
    // 800 KB such a tile takes through the compute unit's memory pipeline otherwise).
    // HC = 0: a wavefront without an item
    const auto own_rows = [&](int w, int& rt_own) {
      const int own_max = (RT + RS - 1) / RS;
      rt_own = w / SG * own_max;
      return RT - rt_own < 0 ? 0 : (RT - rt_own < own_max ? RT - rt_own : own_max);
    };
    GemmPhase<T, NT_O, C, C, NW, RS, 1, true> oproj(reinterpret_cast<const T*>(args->layer.w_o), wave);
    oproj.forget();
    {
      int rt_own;
      if (own_rows(wave, rt_own) > 0) oproj.prefetch();            // in flight during the attention phase
    }
    // The set table, by the first wavefront: it is through with its part of the projection first (the compute unit issues its
    // oldest wavefronts first) and would wait for the others.  (In front of the rows' request every wavefront waits for it: 0.6 k
    // clocks a tile, 4 k with sets of 90 rows and a list of the items instead of this table.)
    if (wave == 0) {
      const int32_t* hdr = header(tab);
      int ns = __builtin_amdgcn_readfirstlane(hdr[1]);
      ns = ns < 0 ? 0 : (ns > kMaxSets ? kMaxSets : ns);
      const int sl = lane & (kSetWords - 1), r0 = hdr[kHdrR0 + sl], nu_w = hdr[kHdrNu + sl];
      constexpr int kNuMax = SETS == kSets48 ? 48 : kTauMax;
      const int nu = nu_w < 1 ? 1 : (nu_w > kNuMax ? kNuMax : nu_w), kts = (nu + 15) >> 4;
      const int cnt = lane < ns ? kts * item_groups(kts, HEADS, big_heads(C, DUP, SETS)) : 0;
      const int incl = half_wave_scan(cnt);
      const bool shared = groups_per_cu<T, C, HEADS, HID>(SETS) > 1 && n_tiles > kComputeUnits;
      const int split = !shared && split_items(__builtin_amdgcn_readlane(incl, kSetWords - 1),
                                               __ballot(lane < ns && kts > split_key_tiles<T, C, HEADS, HID>()) != 0ull, NW) ? 1 : 0;
      if (lane < kSetWords)
        set_tab[lane] = lane < ns ? set_word(r0 < 0 ? 0 : (r0 > kRowsMax - 4 ? kRowsMax - 4 : r0), nu, (incl - cnt) << split) : kNoItem;
      if (lane == kSetWords - 1) { set_tab[kSetWords] = (unsigned)(incl << split); set_tab[kSetWords + 1] = (unsigned)split; }
    } else if (LONG && wave == 1) {
      int then = -1;
      if (n_tiles > kGrid) then = Shares(n_tiles, kGrid).tile(blockIdx.x, stride, __builtin_amdgcn_readfirstlane((int)set_tab[kSetWords + 3]));
      if (lane == 0) set_tab[kSetWords + 2] = (unsigned)then;
    }
    lds_barrier();
    DSVT_REFRESH_LANE();

    if constexpr (LONG) {
      next = __builtin_amdgcn_readfirstlane((int)set_tab[kSetWords + 2]);
      more = next >= 0;
    }
    DSVT_PHASE(tile, 3);                               // Q, K, V^T in LDS
    // ---- 4. attention inside every set; O overwrites Q
    {
      const PositionTable table = {args->layer.rel_bias, args->layer.rel_const, args->layer.rel_last, args->layer.rel_none};
      const unsigned my_set = set_tab[lane & (kSetWords - 1)];
      const int n_items = __builtin_amdgcn_readfirstlane((int)set_tab[kSetWords]), split = __builtin_amdgcn_readfirstlane((int)set_tab[kSetWords + 1]);
      for (int it = wave; it < n_items; it += NW) {
        // (both halves of the wavefront hold the table; set 0 starts at item 0)
        const int s = __popcll(__ballot((int)(my_set >> 16) <= it) & 0xffffffffull) - 1;
        const unsigned sw = (unsigned)__builtin_amdgcn_readlane((int)my_set, s);
        const int r0 = sw & 255, nu = (sw >> 8) & 255, kts = (nu + 15) >> 4, k = it - (int)(sw >> 16);
        const int ngr = item_groups(kts, HEADS, big_heads(C, DUP, SETS)) << split;      // (a power of two)
        const int qt = k >> __builtin_ctz(ngr), hh = k & (ngr - 1);
        attn_any<T, C, HEADS, HID, SETS, DUP>(table, smem, 2 * (int)L::kTile - xo, row_code(tab), row_mult(tab), r0, nu, qt, hh, kts, split != 0, RT * 16);
      }
    }
    // attention is done with V^T behind the next barrier: the GELU table of the MLP and the LayerNorms' scales and shifts
    // take its place (published by the barriers of the LayerNorm below).  Read from memory where they are used, the latter
    // would come back behind the weights requested before them, and the LayerNorm of every wavefront would wait for those.
    // Pass of the 3,001- / 30,000-pillar frame, of the wide windows, of the 120,000-voxel frame: 159.3 -> 156.4, 368.6 ->
    // 365.5, 326 -> 319, 712 -> 707 us.
    constexpr bool kGeluTable = sizeof(T) == 2;
    static_assert(kGeluKnots * sizeof(float2) <= 4096, "GELU table slot");
    constexpr int kGeluThreads = kGeluTable ? kGeluKnots / 2 : 0, kVecThreads = kGeluThreads + C;     // 16 bytes per thread: 4 C floats in C loads
    static_assert(kVecThreads <= NTHREADS, "one load per thread");
    // (Neither the thread number nor a first value of `late` may live through the attention: four zeros kept for it were four
    // registers too many for sets of 49 to 72 voxels of C = 64 with repeats as keys, which spilled eight.)
    DSVT_REFRESH_LANE();
    // (What follows from the wavefront's number is computed anew: kept through the attention, it spills five scalar registers where sets of more than 48
    // voxels are taken, C = 128.)
    int own_wave = wave, rt_own;
    asm volatile("" : "+s"(own_wave));
    const int og_own = own_wave % SG, HC = own_rows(own_wave, rt_own), o_own = og_own * 16 * NT_O;
    f32x4 late;
    opaque_def(late);
    if (full_layer && tid < kVecThreads) {
      const int i = tid - kGeluThreads, v = i / (C / 4);
      const float* src = v < 2 ? (v == 0 ? args->layer.ln1_g : args->layer.ln1_b) : (v == 2 ? args->layer.ln2_g : args->layer.ln2_b);
      late = i < 0 ? reinterpret_cast<const f32x4*>(args->layer.gelu_tab)[tid] : reinterpret_cast<const f32x4*>(src)[i - v * (C / 4)];
    }
    f32x4 bo4[NT_O];
#pragma unroll
    for (int nt = 0; nt < NT_O; ++nt) bo4[nt] = *reinterpret_cast<const f32x4*>(args->layer.b_o + o_own + 16 * nt + 4 * g);
    int next_word;
    opaque_def(next_word);
    if (more && tid < 256) next_word = args->maps.tile_desc[(size_t)next * 256 + tid];
    lds_barrier();
    DSVT_REFRESH_LANE();
    DSVT_PHASE(tile, 4);                               // attention done
    static_assert(L::total < 0x40000 && L::off_gelu % 8 == 0, "gelu_entry's addresses");
    const float* affine_lds = reinterpret_cast<const float*>(smem + L::off_aff);
    if (full_layer && tid < kVecThreads)
      *reinterpret_cast<f32x4*>(smem + (tid < kGeluThreads ? L::off_gelu : L::off_aff - kGeluThreads * 16) + tid * 16) = late;

    // ---- 5. Y = O Wo^T + bo (+ x), then LayerNorm; the result replaces x in Xs (or raw Y goes out)
    // The first MLP matrix is requested during this phase, by a third of the wavefronts at a time
    // (before the projection, after it, after the residual): a CU takes a 16-byte load per
    // wavefront every ~16 cycles, a wavefront waits until its requests are taken, and twelve
    // wavefronts asking at once would all stand still for 3 k cycles.
    GemmPhase<T, NT_1, C, HID, NW, 1, 1, true> ffn1(reinterpret_cast<const T*>(args->layer.w_1), wave);
    const int pf_turn = full_layer ? wave / (NW / 3) : -1;
    ffn1.forget();
    if (pf_turn == 0) ffn1.prefetch();
    f32x4 keep[NT_O][kOwnTiles];
    QkvPhase qkv(reinterpret_cast<const T*>(args->layer.w_qkv), wave);     // of the next tile
    if (HC == 1) oproj.template run_keep<1>(Qs, LDX, rt_own, bo4, keep);
    else if (HC == 2) oproj.template run_keep<2>(Qs, LDX, rt_own, bo4, keep);
    else if (kOwnTiles == 3 && HC == 3) oproj.template run_keep<kOwnTiles>(Qs, LDX, rt_own, bo4, keep);
    else undefined(keep);
    if (pf_turn == 1) ffn1.prefetch();
    if (!full_layer) {                           // attention and its projection only: raw Y goes out, one tile per workgroup
      if constexpr (kPairs) {
        if (HC > 0) put_pair(args->out, tab, R, 16 * rt_own + m, HC > 1, o_own, pack4<T>(keep[0][0]), pack4<T>(keep[0][kOwnTiles - 1]));
      } else {
#pragma unroll
        for (int r = 0; r < kOwnTiles; ++r)
          if (r < HC) {
            f32x4 y[NT_O];
#pragma unroll
            for (int nt = 0; nt < NT_O; ++nt) y[nt] = keep[nt][r];
            put_out(args->out, tab, R, 16 * (rt_own + r) + m, o_own, y);
          }
      }
      return;
    }
    add_rows<T, NT_O, kOwnTiles>(keep, Xs, LDX, rt_own, HC, o_own);
    if (pf_turn == 2) ffn1.prefetch();
    layer_norm_tile<T, NT_O, C, kOwnTiles>(keep, o_own, og_own, rt_own, HC, stat, [&](int nt, f32x4& a, f32x4& b) {
      a = *reinterpret_cast<const f32x4*>(affine_lds + o_own + 16 * nt + 4 * g);
      b = *reinterpret_cast<const f32x4*>(affine_lds + C + o_own + 16 * nt + 4 * g);
    }, args->layer.ln_eps, [&](int, int row, const f32x4 (&y)[NT_O]) {
#pragma unroll
      for (int nt = 0; nt < NT_O; ++nt) *reinterpret_cast<Vec4*>(Xs + row * LDX + o_own + 16 * nt + (4 * g ^ swizzle<T>(m))) = pack4<T>(y[nt]);
    });
    if (more) store_desc(next_word, (int)L::kRowTab - tab, args->maps.n_voxels);
    lds_barrier();
    DSVT_REFRESH_LANE();

    DSVT_PHASE(tile, 5);                             // x1 in LDS
    // ---- 6. MLP: H = gelu(x1 W1^T + b1) over the dead Q/K tiles; x2 = LN(x1 + H W2^T + b2)
    // The second matrix's weights (C = 192: the first half of K, C <= 128: all) are requested between the last MFMAs of the first
    // product and the GELU of its last row tiles: the memory pipeline is idle there and needs 2.7 k cycles for the 144 fragments of
    // C = 192, the GELU of two row tiles and three wavefronts per SIMD about 2 k.  Passes with the request behind the GELU and with it
    // here (two sessions): 3,001-pillar frame 156.4 / 155.7 us, 30,000-pillar frame 365.5 / 361.8, wide windows (C = 128) 319 / 316,
    // 120,000-voxel frame 707 / 699.  Slower than this at C = 192, each in one session with it: the matrix in three slices, two of
    // them requested here, 0.2-0.8 %; the same with the MLP's biases from LDS beside the LayerNorms' vectors 0.6-1.4 %; the second
    // bias requested in front of the weights 0.1-0.7 %.
    GemmPhase<T, NT_2, HID, C, NW, RS, (HID / Mma<T>::KC > 8 ? 2 : 1), true> ffn2(reinterpret_cast<const T*>(args->layer.w_2), wave);
    const float gelu0 = gelu_start(smem + L::off_gelu);
    // Parts of a row tile's epilogue: the table entries of output tile 0, 1, .. requested, then the values of output tile 0, 1, ..
    f32x2 chord[NT_1][4];
    ffn1.template run_before<2 * NT_1>(Xs, LDX, RT, args->layer.b_1, [&](int k, int o0, int r, f32x4 (&acc)[NT_1]) {
      if (kGeluTable && k < NT_1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) chord[k][i] = gelu_entry(gelu0, acc[k][i]);
      }
      if (k >= NT_1 && k < 2 * NT_1) {
        const int nt = k - NT_1;
        f32x4 v = acc[nt];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = kGeluTable ? fmaf(chord[nt][i].x, v[i], chord[nt][i].y) : gelu_erf_fast(v[i]);
        *reinterpret_cast<Vec4*>(Hs + (16 * r + m) * LDH + o0 + 16 * nt + (4 * g ^ swizzle<T>(m))) = pack4<T>(v);
      }
    }, [&]() {
      ffn2.forget();
      if (HC > 0) ffn2.prefetch();
    });
    const int o_own2 = og_own * 16 * NT_2;
    f32x4 b24[NT_2];
#pragma unroll
    for (int nt = 0; nt < NT_2; ++nt) b24[nt] = *reinterpret_cast<const f32x4*>(args->layer.b_2 + o_own2 + 16 * nt + 4 * g);
    // The next tile's rows: in flight during the second product, stored over Q when every wavefront is through with it
    const int next_tab = (int)L::kRowTab - tab, next_RT = more ? row_tiles(tile_rows(next_tab)) : 0;
    uint4 gv[G];
    unsigned live = 0u;
#pragma unroll
    for (int k = 0; k < G; ++k) { opaque_def(gv[k].x); opaque_def(gv[k].y); opaque_def(gv[k].z); opaque_def(gv[k].w); }
    if (more) request_rows(gv, live, next_tab, next_RT, args->x);
    lds_barrier();
    DSVT_REFRESH_LANE();
    DSVT_PHASE(tile, 6);                             // H in LDS
    f32x4 keep2[NT_2][kOwnTiles];
    if (HC == 1) ffn2.template run_keep<1>(Hs, LDH, rt_own, b24, keep2);
    else if (HC == 2) ffn2.template run_keep<2>(Hs, LDH, rt_own, b24, keep2);
    else if (kOwnTiles == 3 && HC == 3) ffn2.template run_keep<kOwnTiles>(Hs, LDH, rt_own, b24, keep2);
    else undefined(keep2);
    qkv.forget();
    if (more && pf_turn == 0) qkv.template prefetch_first<kEarly>();
    add_rows<T, NT_2, kOwnTiles>(keep2, Xs, LDX, rt_own, HC, o_own2);
    if (more && pf_turn == 1) qkv.template prefetch_first<kEarly>();
    Vec4 held;                                   // the first of two row tiles' rows (kPairs)
    opaque_def(held);
    layer_norm_tile<T, NT_2, C, kOwnTiles>(keep2, o_own2, og_own, rt_own, HC, stat, [&](int nt, f32x4& a, f32x4& b) {
      if (nt == 0) DSVT_PHASE(tile, 7);          // everybody's part of the second product done
      if (nt == 0 && more) {
        store_rows(gv, live, 2 * (int)L::kTile - xo, next_RT);
        if (pf_turn == 2) qkv.template prefetch_first<kEarly>();
      }
      a = *reinterpret_cast<const f32x4*>(affine_lds + 2 * C + o_own2 + 16 * nt + 4 * g);
      b = *reinterpret_cast<const f32x4*>(affine_lds + 3 * C + o_own2 + 16 * nt + 4 * g);
    }, args->layer.ln_eps, [&](int r, int row, const f32x4 (&y)[NT_2]) {
      if constexpr (kPairs) {
        if (r == 0) held = pack4<T>(y[0]);
        if (r + 1 == HC) put_pair(args->out, tab, R, row - 16 * r, r > 0, o_own2, held, pack4<T>(y[0]));
      } else {
        put_out(args->out, tab, R, row, o_own2, y);
      }
    });
    DSVT_PHASE(tile, 8);
    if (!more) return;
    DSVT_PHASE(next, 0);
    DSVT_PHASE(next, 1);
    qkv.template prefetch_rest<kEarly>(args->layer.b_qkv, 2 * C / (16 * NT_QKV));
    tile = next;
    stride = LONG ? stride + 1 : 2 * (int)gridDim.x - stride;
    xo = 2 * (int)L::kTile - xo;
    tab = (int)L::kRowTab - tab;
    R = tile_rows(tab);
    RT = row_tiles(R);
    lds_barrier();
    DSVT_REFRESH_LANE();
    DSVT_PHASE(tile, 2);
    project(qkv, RT);
  }
}

template <typename T, int C, int HEADS, int HID, int NT_QKV, int NT_O, int NT_1, int NT_2, SetSize SETS, bool DUP>
__global__ void __launch_bounds__(kLayerWaves * 64, (3 * groups_per_cu<T, C, HEADS, HID>(SETS)))
k_layer(LayerCall<T> call) { layer_tiles<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, SETS, DUP, false>(call); }
// The same for frames of several rounds of tiles.
template <typename T, int C, int HEADS, int HID, int NT_QKV, int NT_O, int NT_1, int NT_2, SetSize SETS, bool DUP>
__global__ void __launch_bounds__(kLayerWaves * 64, (3 * groups_per_cu<T, C, HEADS, HID>(SETS)))
k_long_layer(LayerCall<T> call) { layer_tiles<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, SETS, DUP, true>(call); }

// ------------------------------------------------------------------------------------------
// Packed buffer of a layer: the four matrices in fragment order, each on a 256-byte boundary.
struct PackedLayout { size_t off[6], total; int out[4], k[4]; int rel_size; };   // off[4]: position table, off[5]: GELU table
PackedLayout packed_layout(const dsvt_layer_w& w) {
  PackedLayout pl;
  const size_t es = w.dtype == DSVT_BF16 ? 2 : 4;
  const int out[4] = {3 * w.C, w.C, w.hidden, w.C}, k[4] = {w.C, w.C, w.C, w.hidden};
  size_t o = 0;
  for (int i = 0; i < 4; ++i) { pl.off[i] = o; pl.out[i] = out[i]; pl.k[i] = k[i]; o = dsvt_align_up(o + (size_t)out[i] * k[i] * es, 256); }
  // position table [heads / 4][index][4] plus one last row of -inf each (the row of a key that does not exist); without a
  // positional term the table is one row of zeros and that last row
  pl.rel_size = w.rel_bias != nullptr ? (2 * w.win[0] - 1) * (2 * w.win[1] - 1) * (2 * w.win[2] - 1) : 1;
  pl.off[4] = o;
  o = dsvt_align_up(o + (size_t)(pl.rel_size + 1) * w.heads * 4, 256);
  pl.off[5] = o;
  o = dsvt_align_up(o + (size_t)kGeluKnots * sizeof(float2), 256);
  pl.total = o;
  return pl;
}

// [heads][size] -> [heads / 4][size + 1][4], in units of log2(e) (the softmax works with exp2); row `size` holds -inf.
// src == nullptr (no positional term): zeros.
__global__ void k_pack_table(const float* __restrict__ src, float* __restrict__ dst, int heads, int size) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= heads * (size + 1)) return;
  const int h = i / (size + 1), k = i - h * (size + 1);
  dst[((size_t)(h / 4) * (size + 1) + k) * 4 + h % 4] = k == size ? -INFINITY : (src != nullptr ? src[(size_t)h * size + k] * 1.4426950408889634f : 0.f);
}

LayerDev to_dev(const dsvt_layer_w& w) {
  LayerDev d;
  const PackedLayout pl = packed_layout(w);
  const char* pk = reinterpret_cast<const char*>(w.packed);
  d.w_qkv = pk + pl.off[0]; d.w_o = pk + pl.off[1]; d.w_1 = pk + pl.off[2]; d.w_2 = pk + pl.off[3];
  d.b_qkv = w.b_qkv; d.b_o = w.b_o; d.b_1 = w.b_1; d.b_2 = w.b_2;
  d.ln1_g = w.ln1_g; d.ln1_b = w.ln1_b; d.ln2_g = w.ln2_g; d.ln2_b = w.ln2_b;
  d.rel_bias = reinterpret_cast<const float*>(pk + pl.off[4]);
  d.gelu_tab = reinterpret_cast<const float2*>(pk + pl.off[5]);
  d.ln_eps = w.ln_eps;
  const int my = 2 * w.win[1] - 1, mz = 2 * w.win[2] - 1;
  d.rel_my = my; d.rel_mz = mz;
  constexpr unsigned row = kRelRow;
  d.rel_last = (unsigned)(pl.rel_size - 1) * row;
  d.rel_none = (unsigned)pl.rel_size * row;
  d.rel_const = w.rel_bias != nullptr ? (unsigned)(((w.win[0] - 1) * my + (w.win[1] - 1)) * mz + (w.win[2] - 1)) * row : 0u;
  return d;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_layer(const dsvt_layer_w& w, bool need_mlp, bool need_packed = true) {
  if (!w.w_qkv || !w.w_o || !w.b_qkv || !w.b_o) return DSVT_EINVAL;
  if (need_packed && (!w.packed || !aligned16(w.packed))) return DSVT_EINVAL;
  if (need_mlp && (!w.w_1 || !w.w_2 || !w.b_1 || !w.b_2 || !w.ln1_g || !w.ln1_b || !w.ln2_g || !w.ln2_b)) return DSVT_EINVAL;
  if (w.dtype != DSVT_F32 && w.dtype != DSVT_BF16) return DSVT_EINVAL;
  if (w.dup_mode != 0 && w.dup_mode != 1) return DSVT_EINVAL;
  for (int a = 0; a < 3; ++a) if (w.win[a] <= 0) return DSVT_EINVAL;
  if (!((w.C == 64 && w.heads == 4 && w.hidden == 128) || (w.C == 128 && w.heads == 8 && w.hidden == 256) ||
        (w.C == 192 && w.heads == 8 && w.hidden == 384)))
    return DSVT_EUNSUPPORTED;
  if (w.dtype == DSVT_F32 && w.C != 64) return DSVT_EUNSUPPORTED;   // wider fp32 tiles exceed the 160 KB LDS
  const void* ptrs[] = {w.w_qkv, w.w_o, w.w_1, w.w_2, w.b_qkv, w.b_o, w.b_1, w.b_2, w.ln1_g, w.ln1_b, w.ln2_g, w.ln2_b};
  for (const void* q : ptrs) if (q && !aligned16(q)) return DSVT_EINVAL;
  return DSVT_OK;
}

int check_maps(const dsvt_maps& mp) {
  if (!mp.set_inds || !mp.n_sets || mp.n_voxels <= 0 || mp.max_sets <= 0 || mp.tau <= 0) return DSVT_EINVAL;
  if (mp.tau > kTauMax) return DSVT_EUNSUPPORTED;
  if (mp.tiles.tile_desc == nullptr && mp.tau > 64) return DSVT_EUNSUPPORTED;   // without a work list a wavefront scans a set's tau slots
  const dsvt_tile_list& tl = mp.tiles;
  const bool any = tl.tile_first || tl.n_tiles || tl.tile_order || tl.tile_desc;
  const bool all = tl.tile_first && tl.n_tiles && tl.tile_order && tl.tile_desc;
  if (any && (!all || tl.max_tiles <= 0)) return DSVT_EINVAL;
  return DSVT_OK;
}

template <typename T, int C, int HEADS, int HID, int NT_QKV, int NT_O, int NT_1, int NT_2, SetSize SETS, bool DUP, bool LONG = false>
int launch_layer_v(const dsvt_layer_w& w, const dsvt_maps& mp, const int32_t* coords, const void* x, void* out, int full,
                   hipStream_t st) {
  const auto kernel = []() {
    if constexpr (LONG) return k_long_layer<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, SETS, DUP>;
    else return k_layer<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, SETS, DUP>;
  };
  auto kern = kernel();
  constexpr size_t lds = LayerLds<T, C, HEADS, HID>::total;
  static std::atomic<uint64_t> lds_allowed{0};
  if (int rc = dsvt_allow_lds(reinterpret_cast<const void*>(kern), lds, lds_allowed)) return rc;
  MapsDev md;
  md.set_inds = mp.set_inds; md.n_sets = mp.n_sets; md.n_tiles = mp.tiles.n_tiles; md.tile_desc = mp.tiles.tile_desc;
  md.max_sets = mp.max_sets; md.max_tiles = mp.tiles.max_tiles; md.tau = mp.tau; md.n_voxels = mp.n_voxels;
  const int64_t tiles = mp.tiles.tile_desc ? mp.tiles.max_tiles : dsvt_ceil_div(mp.max_sets, fixed_sets(mp.tau));
  constexpr int64_t fit = kComputeUnits * groups_per_cu<T, C, HEADS, HID>(SETS);
  const unsigned grid = (unsigned)(full && mp.tiles.tile_desc && tiles > fit ? fit : tiles);
  dsvt_prof_scope ps(DSVT_K_LAYER, st);
  const LayerCall<T> call = {to_dev(w), md, reinterpret_cast<const int4*>(coords), reinterpret_cast<const T*>(x), reinterpret_cast<T*>(out), full};
  kern<<<grid, kLayerWaves * 64, lds, st>>>(call);
  return DSVT_OK;
}

// Whether sets of 49 voxels and more take kSets96Slim, where a tile leaves room in the LDS for a second workgroup on the
// compute unit (C = 64 in bf16): it also leaves room in the registers (67 of them, 74 with repeats as keys; kSets96: 96 and
// 104), which pays once there are more tiles than compute units -- about max(48, 5 / 6 tau) voxels a tile --; with larger sets,
// fetching the table rows once for two heads is worth as much.  Two layers, kSets96 -> slim (repeats as keys within 0.9 us of
// these).  30 x 30 windows, sets of up to 50 voxels: 12,000 voxels 20.0 -> 21.9 us, 12,800 29.6 -> 25.6, 20,000 31.8 -> 29.1, 40,000 57.7 -> 46.4; up
// to 64: 13,568 21.6 -> 24.5, 14,000 29.9 -> 28.3, 20,000 34.4 -> 32.9, 40,000 51.8 -> 52.2; up to 72: 15,000 23.5 -> 28.4, 16,000
// 31.6 -> 32.9, 20,000 34.9 -> 36.9, 40,000 53.9 -> 56.9; up to 80: 18,000 32.4 -> 34.7, 40,000 57.6 -> 62.5.  24 x 24 windows, up to 60: 25,000
// 34.5 -> 32.5, 40,000 59.1 -> 46.3; up to 72: 25,000 35.2 -> 36.7, 40,000 52.5 -> 50.2, 60,000 71.7 -> 68.0.  Without a work list, 12 x 12 windows,
// up to 50 to 64, slim takes a third less throughout.  So the line could lie at 64 where windows are full; and a frame whose tiles, few voxels over the
// line, still fit the compute units once loses up to a fifth: 18,000 voxels in 24 x 24 windows, up to 60: 23.5 -> 28.2.  (The number of tiles is not known on the host.)
bool slim_sets(const dsvt_maps& mp) {
  const int per_tile = 5 * mp.tau / 6 > 48 ? 5 * mp.tau / 6 : 48;
  return mp.tau <= 72 && mp.n_voxels > 256 * per_tile;
}

// Whole layers with a work list of at least two full rounds of tiles (a tile has at most 96 rows), sets of up to 48 voxels.  Where the number
// of tiles does not follow from that of the voxels -- 41,000 pillars have 656 to 722 -- going back and forth through the list is within 1.5 % of it,
// and finding the tiles costs a layer of a single round up to 1 %.
template <typename T, int C, int HEADS, int HID>
bool is_long(const dsvt_maps& mp, int full) {
  return full && mp.tiles.tile_desc && mp.n_voxels > kRowsMax * 2 * kComputeUnits * groups_per_cu<T, C, HEADS, HID>(kSets48);
}

template <typename T, int C, int HEADS, int HID, int NT_QKV, int NT_O, int NT_1, int NT_2>
int launch_layer(const dsvt_layer_w& w, const dsvt_maps& mp, const int32_t* coords, const void* x, void* out, int full,
                 hipStream_t st) {
  // instantiations per range of set sizes and reading of repeated slots: as keys (dup_mode 1) they multiply the
  // exponentials by the slots' counts
  constexpr bool kSlim = two_groups_fit<T, C, HEADS, HID>();
  const bool dup = w.dup_mode != 0;
  if (mp.tau <= 48) {
    if (is_long<T, C, HEADS, HID>(mp, full)) {
      if (dup) return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets48, true, true>(w, mp, coords, x, out, full, st);
      return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets48, false, true>(w, mp, coords, x, out, full, st);
    }
    if (dup) return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets48, true>(w, mp, coords, x, out, full, st);
    return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets48, false>(w, mp, coords, x, out, full, st);
  }
  if constexpr (kSlim) {
    if (slim_sets(mp)) {
      if (dup) return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets96Slim, true>(w, mp, coords, x, out, full, st);
      return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets96Slim, false>(w, mp, coords, x, out, full, st);
    }
  }
  if (dup) return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets96, true>(w, mp, coords, x, out, full, st);
  return launch_layer_v<T, C, HEADS, HID, NT_QKV, NT_O, NT_1, NT_2, kSets96, false>(w, mp, coords, x, out, full, st);
}

int run_layer(const dsvt_layer_w& w, const dsvt_maps& mp, const int32_t* coords, const void* x, void* out, int full,
              hipStream_t st) {
  if (w.dtype == DSVT_BF16) {
    if (w.C == 192) return launch_layer<bf16_t, 192, 8, 384, 3, 2, 2, 2>(w, mp, coords, x, out, full, st);
    if (w.C == 128) return launch_layer<bf16_t, 128, 8, 256, 2, 2, 2, 2>(w, mp, coords, x, out, full, st);
    return launch_layer<bf16_t, 64, 4, 128, 1, 1, 1, 1>(w, mp, coords, x, out, full, st);
  }
  return launch_layer<float, 64, 4, 128, 1, 1, 1, 1>(w, mp, coords, x, out, full, st);
}

}  // namespace


extern "C" int dsvt_layer_packed_size(const dsvt_layer_w* layer, size_t* bytes) {
  if (!layer || !bytes) return DSVT_EINVAL;
  int rc = check_layer(*layer, true, false);
  if (rc != DSVT_OK) return rc;
  *bytes = packed_layout(*layer).total;
  return DSVT_OK;
}

extern "C" int dsvt_layer_pack(const dsvt_layer_w* layer, void* packed, size_t bytes, void* stream) {
  if (!layer || !packed || !aligned16(packed)) return DSVT_EINVAL;
  int rc = check_layer(*layer, true, false);
  if (rc != DSVT_OK) return rc;
  const PackedLayout pl = packed_layout(*layer);
  if (bytes < pl.total) return DSVT_ENOSPC;
  const void* src[4] = {layer->w_qkv, layer->w_o, layer->w_1, layer->w_2};
  hipStream_t st = (hipStream_t)stream;
  for (int i = 0; i < 4; ++i) {
    char* dst = reinterpret_cast<char*>(packed) + pl.off[i];
    if (layer->dtype == DSVT_BF16) {
      const long long slots = (long long)(pl.out[i] / 16) * (pl.k[i] / Mma<bf16_t>::KC) * 64;
      k_pack<bf16_t><<<(unsigned)dsvt_ceil_div(slots, 256), 256, 0, st>>>(reinterpret_cast<const bf16_t*>(src[i]),
                                                                        reinterpret_cast<bf16_t*>(dst), pl.out[i], pl.k[i]);
    } else {
      const long long slots = (long long)(pl.out[i] / 16) * (pl.k[i] / Mma<float>::KC) * 64;
      k_pack<float><<<(unsigned)dsvt_ceil_div(slots, 256), 256, 0, st>>>(reinterpret_cast<const float*>(src[i]),
                                                                       reinterpret_cast<float*>(dst), pl.out[i], pl.k[i]);
    }
  }
  k_pack_gelu_table<<<(unsigned)dsvt_ceil_div(kGeluKnots, 256), 256, 0, st>>>(
      reinterpret_cast<float2*>(reinterpret_cast<char*>(packed) + pl.off[5]));
  {
    const int n = (pl.rel_size + 1) * layer->heads;
    k_pack_table<<<(unsigned)dsvt_ceil_div(n, 256), 256, 0, st>>>(
        layer->rel_bias, reinterpret_cast<float*>(reinterpret_cast<char*>(packed) + pl.off[4]), layer->heads, pl.rel_size);
  }
  DSVT_HIP_TRY(hipGetLastError());
  return DSVT_OK;
}

extern "C" int dsvt_set_attention_workspace_size(const dsvt_layer_w* layer, int32_t n_voxels, size_t* bytes) {
  if (!layer || !bytes || n_voxels <= 0) return DSVT_EINVAL;
  *bytes = 0;
  return DSVT_OK;
}

extern "C" int dsvt_block_workspace_size(const dsvt_layer_w* layer, int32_t n_voxels, size_t* bytes) {
  if (!layer || !bytes || n_voxels <= 0) return DSVT_EINVAL;
  *bytes = 0;
  return DSVT_OK;
}

extern "C" int dsvt_set_attention(const dsvt_layer_w* layer, const dsvt_maps* maps, const int32_t* coords,
                                  const void* x, void* y, void* ws, size_t ws_bytes, void* stream) {
  (void)ws; (void)ws_bytes;
  if (!layer || !maps || !coords || !x || !y || x == y) return DSVT_EINVAL;
  int rc = check_layer(*layer, false);
  if (rc != DSVT_OK) return rc;
  rc = check_maps(*maps);
  if (rc != DSVT_OK) return rc;
  if (!aligned16(x) || !aligned16(y) || !aligned16(coords)) return DSVT_EINVAL;
  rc = run_layer(*layer, *maps, coords, x, y, 0, (hipStream_t)stream);
  if (rc != DSVT_OK) return rc;
  DSVT_HIP_TRY(hipGetLastError());
  return DSVT_OK;
}

extern "C" int dsvt_block(const dsvt_layer_w layer[2], const dsvt_maps maps[2], const int32_t* coords,
                          const void* x_in, void* x_out, void* ws, size_t ws_bytes, void* stream) {
  (void)ws; (void)ws_bytes;
  if (!layer || !maps || !coords || !x_in || !x_out) return DSVT_EINVAL;
  for (int l = 0; l < 2; ++l) {
    int rc = check_layer(layer[l], true);
    if (rc != DSVT_OK) return rc;
    rc = check_maps(maps[l]);
    if (rc != DSVT_OK) return rc;
    if (layer[l].C != layer[0].C || layer[l].dtype != layer[0].dtype || maps[l].n_voxels != maps[0].n_voxels)
      return DSVT_EINVAL;
  }
  if (!aligned16(x_in) || !aligned16(x_out) || !aligned16(coords)) return DSVT_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const void* src = x_in;
  for (int l = 0; l < 2; ++l) {
    int rc = run_layer(layer[l], maps[l], coords, src, x_out, 1, st);
    if (rc != DSVT_OK) return rc;
    src = x_out;
  }
  DSVT_HIP_TRY(hipGetLastError());
  return DSVT_OK;
}
