// MFMA building blocks for gfx950 (64-lane wavefronts).
//
// All dense contractions of the path are skinny GEMMs  Out^T[o][r] = sum_k W[o][k] * X[r][k]:
// the weight matrix W ([out,in], in global memory, cache resident) is the MFMA "A" operand and
// the activations X ([rows, features], staged in LDS) are the "B" operand.  With 16x16 output
// tiles lane l = 16*g + m holds
//     A fragment: row m of the tile, the k-slice owned by lane group g (16 contiguous bytes)
//     B fragment: column m of the tile, the same k-slice                (16 contiguous bytes)
//     accumulator: acc[i] = Out^T[4*g + i][m]  -- four consecutive output features of one row,
// so results go back to a [rows, features] LDS tile with one vector store per lane and can be
// the B operand of the next contraction without a transpose.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16_t;
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mma;

// bf16: one v_mfma_f32_16x16x32_bf16 per fragment pair; a lane owns 8 consecutive k.
template <> struct Mma<bf16_t> {
  typedef bf16x8 Frag;
  typedef bf16x4 Vec4;                 // four values = one accumulator's worth, 8 bytes
  static constexpr int KC = 32;        // k extent of a fragment over the whole wavefront
  static constexpr int KL = 8;         // k per lane
  static __device__ __forceinline__ f32x4 mma(Frag a, Frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// fp32: four v_mfma_f32_16x16x4_f32 per fragment pair; a lane owns 4 consecutive k and step e of
// the four consumes element e of every lane (the k order inside a fragment is irrelevant as long
// as A and B agree, which they do).
template <> struct Mma<float> {
  typedef f32x4 Frag;
  typedef f32x4 Vec4;
  static constexpr int KC = 16;
  static constexpr int KL = 4;
  static __device__ __forceinline__ f32x4 mma(Frag a, Frag b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], c, 0, 0, 0);
    return c;
  }
};

template <typename T> __device__ __forceinline__ typename Mma<T>::Vec4 pack4(f32x4 v);
template <> __device__ __forceinline__ bf16x4 pack4<bf16_t>(f32x4 v) {
  bf16x4 r = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
  return r;
}
template <> __device__ __forceinline__ f32x4 pack4<float>(f32x4 v) { return v; }

template <typename T> __device__ __forceinline__ float to_f32(T v) { return (float)v; }

// threadIdx.x behind an empty asm: values derived from it (lane, row and feature offsets) are
// recomputed where they are used -- a couple of ALU instructions -- instead of being kept in
// registers from the top of a long kernel, where they end up spilled to scratch memory (and a
// reload from scratch waits for every outstanding global load, the weights requested ahead).
__device__ __forceinline__ int opaque_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Declares v defined, with whatever its registers hold and without an instruction.  For variables that are assigned
// on some paths only and read on those paths only: in a loop, the compiler otherwise moves the "undefined" definition
// of the other paths in front of the loop and keeps registers for it through every iteration.
template <typename V> __device__ __forceinline__ void opaque_def(V& v) { asm volatile("" : "=v"(v)); }

template <int A, int B> __device__ __forceinline__ void undefined(f32x4 (&v)[A][B]) {
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) opaque_def(v[a][b]);
}

// Elements of T that pad every LDS row by 32 bytes.  Rows of K elements (K * sizeof(T) a multiple
// of 64 bytes) then have a pitch that is an odd multiple of 32 bytes, the one pitch at which the
// 16-byte fragment loads of a wavefront (16 rows x 4 k-slices) run at the full LDS rate; measured
// on gfx950: 225 B/clk per CU against 125-150 B/clk for pitches of 16, 48 or 0 mod 64 bytes.
template <typename T> constexpr int lds_pad() { return 32 / (int)sizeof(T); }

// Swizzled rows: in every other group of four rows the two 16-byte pieces of each 32 bytes change places.  At that pitch the 8-byte stores of
// accumulators (16 rows, one place in each) hit a bank four times, since a store sees 32 banks: 16.1 clocks an instruction; swizzled they
// hit it twice, 8.2, and the fragment loads stay at their 4.0 (for stores alone an odd multiple of 8 bytes would be best, 6.4, but loads of 16 bytes take
// 8.0 there).  Without -> with: a 64-row tile of C = 192 35.8 -> 35.3 k clocks (first MLP matrix 7.03 -> 6.56 k), an 82-row tile 42.9 -> 42.0 k; passes of
// 30,000 pillars 321.3 -> 319.3 us, windows of 12 and 24 cells 454.3 -> 449.1, 30 x 30 windows 243.8 -> 242.5, 120,000 voxels 609.0 -> 606.9, 3,001
// pillars and an fp32 block no difference.  Element of T in its row: e ^ swizzle<T>(row).  The pitch and all row starts are multiples of 32 bytes, so an address is swizzled like that too.
template <typename T> __device__ __forceinline__ constexpr int swizzle(int row) { return (row >> 2 & 1) * (16 / (int)sizeof(T)); }

// Packed weights.  A matrix W [OUT, K] is stored fragment by fragment in the order the MFMA "A"
// operand wants it: fragment (tile, kf) -- output rows 16*tile .. +15, k in [kf*KC, (kf+1)*KC) --
// is 1 KB, lane l's 16 bytes at offset 16*l, fragments ordered [tile][kf].  A wavefront's load of
// one fragment is then one fully coalesced 1 KB read (the [out, in] layout would touch 16 rows
// of 64 bytes each, which the L1/L2 path serves about 3x slower).

// Workgroup barrier for data exchanged through LDS: waits for this wavefront's LDS operations
// only.  __syncthreads() also drains the outstanding global loads (on this target loads and
// stores share one counter, and its release fence waits for stores), which would turn every
// barrier into a wait for the weight fragments requested ahead for the following phase.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A-operand fragments of NT output tiles over the whole K, kept in registers: every weight
// fragment is loaded from memory once per workgroup tile and reused for all its rows.
template <typename T, int NT, int NKF> struct AFull { typename Mma<T>::Frag f[NKF][NT]; };
// B-operand fragments of one row tile (16 rows) over the whole K.
template <typename T, int NKF> struct BRow { typename Mma<T>::Frag f[NKF]; };

// Wp: packed matrix with NKF_ALL = K / KC fragments per tile; tiles tile0 + NT0 .. tile0 + NT1 - 1 into their places of
// tiles tile0 .. tile0 + NT - 1, k-fragments kf0 .. kf0 + NKF - 1.
template <typename T, int NT, int NKF, int NKF_ALL, int NT0, int NT1>
__device__ __forceinline__ void load_a_tiles(AFull<T, NT, NKF>& a, const T* __restrict__ Wp, int tile0, int kf0 = 0) {
  typedef typename Mma<T>::Frag Frag;
  const int lane = opaque_tid() & 63;
  const Frag* fp = reinterpret_cast<const Frag*>(Wp) + ((size_t)tile0 * NKF_ALL + kf0) * 64 + lane;
#pragma unroll
  for (int nt = NT0; nt < NT1; ++nt)
#pragma unroll
    for (int kf = 0; kf < NKF; ++kf) a.f[kf][nt] = fp[(nt * NKF_ALL + kf) * 64];
}
template <typename T, int NT, int NKF, int NKF_ALL = NKF>
__device__ __forceinline__ void load_a(AFull<T, NT, NKF>& a, const T* __restrict__ Wp, int tile0, int kf0 = 0) {
  load_a_tiles<T, NT, NKF, NKF_ALL, 0, NT>(a, Wp, tile0, kf0);
}

// Xs: LDS [rows][ldx]; row tile r, k from k0.
template <typename T, int NKF>
__device__ __forceinline__ void load_b(BRow<T, NKF>& b, const T* Xs, int ldx, int r, int k0 = 0) {
  typedef typename Mma<T>::Frag Frag;
  const int lane = opaque_tid() & 63, m = lane & 15, g = lane >> 4;
  const T* xp = Xs + (16 * r + m) * ldx + k0 + g * Mma<T>::KL;
#pragma unroll
  for (int kf = 0; kf < NKF; ++kf) b.f[kf] = *reinterpret_cast<const Frag*>(xp + kf * Mma<T>::KC);
}

template <typename T, int NT, int NKF>
__device__ __forceinline__ void mma_row(f32x4 (&acc)[NT], const AFull<T, NT, NKF>& a, const BRow<T, NKF>& b) {
#pragma unroll
  for (int kf = 0; kf < NKF; ++kf)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = Mma<T>::mma(a.f[kf][nt], b.f[kf], acc[nt]);
}

constexpr int kRowTiles = 6;                     // row tiles of a workgroup tile
constexpr int kRowsMax = 16 * kRowTiles;         // 96 rows
constexpr int kWaves = 8;                        // wavefronts of a pooling workgroup, two per SIMD
constexpr int kKeepRing = 4;                     // see GemmPhase::run_keep() (six fragments spill at C = 192; three and five: no difference)
constexpr int kStatGroupsMax = 6;                // LayerNorm phases: the C features are split over at most 6 groups of output tiles

// One GEMM phase of a workgroup of NW wavefronts: Out^T[NOUT x rows] = W[NOUT x K] . X^T.
// A work item is a group of NT output tiles over all row tiles (RSPLIT = 1) or over one of RSPLIT parts of them; wavefront w
// takes items w, w + NW, ...  run() knows all row tiles and halves (two wavefronts per SIMD), run_keep() any parts of one item
// per wavefront, run_rows() and run_before() one item per wavefront over all row tiles.  An item's weight fragments sit in
// registers for the whole item, run() requests the next item's before the current one is consumed, and the activations of
// row tile r + 1 are read from LDS while row tile r is in the matrix cores.  Every activation
// fragment read from LDS feeds NT MFMAs; a weight fragment is loaded by RSPLIT wavefronts.
// SWZ: the rows of the activations are swizzled (run() reads them as they are and refuses it).
template <typename T, int NT, int K, int NOUT, int NW, int RSPLIT = 1, int KSPLIT = 1, bool SWZ = false>
struct GemmPhase {
  static __device__ __forceinline__ int lane_piece(int lane) { return ((lane >> 4) * Mma<T>::KL) ^ (SWZ ? swizzle<T>(lane & 15) : 0); }
  static constexpr int KC = Mma<T>::KC;
  static constexpr int NKF_ALL = K / KC;
  static constexpr int NKF = NKF_ALL / KSPLIT;          // fragments held at a time (KSPLIT > 1: run_keep only)
  static constexpr int N_OG = NOUT / (16 * NT);
  static constexpr int N_ITEMS = RSPLIT * N_OG;
  static constexpr int IPW = (N_ITEMS + NW - 1) / NW;   // items per wavefront (the last round may be partial)
  static constexpr int RH = kRowTiles / RSPLIT;          // row tiles an item can cover
  static_assert(K % KC == 0 && NOUT % (16 * NT) == 0 && kRowTiles % RSPLIT == 0, "phase shape");
  AFull<T, NT, NKF> a[IPW > 1 ? 2 : 1];                 // two: the next item's weights load during the current item
  const T* Wp;
  int wave;
  struct Bias { f32x4 v[NT]; };                         // an item's bias, see load_bias()
  Bias bias0;                                            // run_rows(): the bias that prefetch_rest() fetched

  __device__ __forceinline__ GemmPhase(const T* wp, int wave_) : Wp(wp), wave(wave_) {}

  // In a loop that requests the weights anew in every trip: called at the top of the trip, it ends the life of the
  // weight registers of the trip before (see opaque_def).
  __device__ __forceinline__ void forget() {
#pragma unroll
    for (int k = 0; k < (int)(sizeof(a) / sizeof(a[0])); ++k)
#pragma unroll
      for (int kf = 0; kf < NKF; ++kf)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) opaque_def(a[k].f[kf][nt]);
  }

  // Request the weights of this wavefront's first item (may be called long before run()).
  __device__ __forceinline__ void prefetch() {
    if (N_ITEMS >= NW || wave < N_ITEMS) load_a<T, NT, NKF, NKF_ALL>(a[0], Wp, (wave % N_OG) * NT);
  }

  // prefetch() in two parts: the first N output tiles of the first item, then the others and the bias run_rows() starts it from.
  template <int N> __device__ __forceinline__ void prefetch_first() {
    if (N_ITEMS >= NW || wave < N_ITEMS) load_a_tiles<T, NT, NKF, NKF_ALL, 0, N>(a[0], Wp, (wave % N_OG) * NT);
  }
  template <int N> __device__ __forceinline__ void prefetch_rest(const float* __restrict__ bias, int swap_og) {
    if (N_ITEMS >= NW || wave < N_ITEMS) {
      load_a_tiles<T, NT, NKF, NKF_ALL, N, NT>(a[0], Wp, (wave % N_OG) * NT);
      load_bias(bias0, bias, wave % N_OG, wave % N_OG >= swap_og);
    }
  }

  // Accumulator start values of output group og: feature 16*nt + 4*g + i for element i, or, with exchanged operands ("sw",
  // wave-uniform), feature 16*nt + m for all four: then element 0 is loaded, and start_bias(), called where the item starts, spreads it.
  __device__ __forceinline__ void load_bias(Bias& b, const float* __restrict__ bias, int og, bool sw) const {
    const int tl = opaque_tid(), lane16 = tl & 15, g4 = ((tl & 63) >> 4) * 4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) opaque_def(b.v[nt]);
    if (sw) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) b.v[nt][0] = bias[og * 16 * NT + 16 * nt + lane16];
    } else {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) b.v[nt] = *reinterpret_cast<const f32x4*>(bias + og * 16 * NT + 16 * nt + g4);
    }
  }
  static __device__ __forceinline__ void start_bias(f32x4 (&b4)[NT], const Bias& b, bool sw) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) b4[nt] = b.v[nt];
    if (sw) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) b4[nt] = f32x4{b4[nt][0], b4[nt][0], b4[nt][0], b4[nt][0]};
    }
  }

  // Row tiles in a rolled loop, two per trip.  epi(o0, r, acc): acc[nt][i] is output
  // feature o0 + 16*nt + 4*g + i of row 16*r + m, bias included.  The bias is fetched before the next item's weights are
  // requested, so waiting for it never waits for them.
  template <typename Epi>
  __device__ __forceinline__ void run(const T* Xs, int ldx, int RT, const float* __restrict__ bias, Epi epi) {
    static_assert(KSPLIT == 1 && (RSPLIT == 1 || RSPLIT == 2), "run() holds the whole K, and an item takes all row tiles or halves");
    static_assert(!SWZ, "run() reads rows that are not swizzled");
    const int h0 = RSPLIT == 1 ? RT : (RT + 1) >> 1;
#pragma unroll
    for (int it = 0; it < IPW; ++it) {
      const int item = wave + it * NW;
      if (item >= N_ITEMS) break;
      const int og = item % N_OG, half = item / N_OG;
      const int rt0 = half ? h0 : 0, cnt = half ? RT - h0 : h0;
      Bias bl;
      load_bias(bl, bias, og, false);
      if (it + 1 < IPW && item + NW < N_ITEMS) load_a<T, NT, NKF>(a[(it + 1) & 1], Wp, ((item + NW) % N_OG) * NT);
      const AFull<T, NT, NKF>& A = a[it & 1];
      if constexpr (RSPLIT == 2) {
        // two wavefronts per SIMD: the other one covers the LDS latency, so one row tile at a
        // time keeps the registers for the second weight buffer
        for (int r = 0; r < cnt; ++r) {
          BRow<T, NKF> b0;
          load_b<T, NKF>(b0, Xs, ldx, rt0 + r);
          f32x4 acc0[NT];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc0[nt] = bl.v[nt];
          mma_row<T, NT, NKF>(acc0, A, b0);
          epi(og * 16 * NT, rt0 + r, acc0);
        }
      } else {
        BRow<T, NKF> b0, b1;
        if (cnt > 0) load_b<T, NKF>(b0, Xs, ldx, rt0);
        for (int r = 0; r < cnt; r += 2) {
          const bool two = r + 1 < cnt;
          if (two) load_b<T, NKF>(b1, Xs, ldx, rt0 + r + 1);
          f32x4 acc0[NT], acc1[NT];              // the bias is the accumulators' initial value
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) { acc0[nt] = bl.v[nt]; acc1[nt] = bl.v[nt]; }
          mma_row<T, NT, NKF>(acc0, A, b0);
          if (two) {
            if (r + 2 < cnt) load_b<T, NKF>(b0, Xs, ldx, rt0 + r + 2);
            mma_row<T, NT, NKF>(acc1, A, b1);
          }
          epi(og * 16 * NT, rt0 + r, acc0);
          if (two) epi(og * 16 * NT, rt0 + r + 1, acc1);
        }
      }
    }
  }

  // (SWAPPED: operands exchanged.  The activations are the MFMA "A" operand and the weights "B" -- their fragment layouts are identical --, so
  // acc[nt][i] = Out[row 4*g + i][feature 16*nt + m]: a lane holds four consecutive rows of one feature, what a transposed store of the result wants.)
  // One row tile, k-fragment by k-fragment: its MFMAs, the same fragment of the row tile at `next` (this lane's piece of it)
  // into the registers just read, then part kf of what the caller has to do meanwhile.  The order is fixed: left to
  // itself the compiler reads a fragment right in front of its MFMAs to save registers, and every one of them waits for LDS.
  // Two row tiles a trip, fragments and table entries where the compiler puts them -> this and run_keep() as it is now: clocks of a 64-row
  // tile of C = 192 38.6 k -> 37.2 k (Q/K/V 6.8 -> 6.3 k, second MLP matrix 5.6 -> 5.1 k, first one 7.25 -> 7.0 k), of an 82-row tile 46.2 -> 44.4 k;
  // passes of 3,001 pillars 146.0 -> 141.8 us, 30,000 339.5 -> 331.4, four frames 1,067 -> 1,030, 30 x 30 windows 273.7 -> 265.6,
  // 120,000 voxels 647.7 -> 631.3, skewed batch 7,217 -> 7,158.
  template <bool SWAPPED, typename Part>
  __device__ __forceinline__ void row_step(f32x4 (&acc)[NT], const f32x4 (&start)[NT], BRow<T, NKF>& b, const T* next, Part part) const {
#pragma unroll
    for (int kf = 0; kf < NKF; ++kf) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const f32x4 c = kf == 0 ? start[nt] : acc[nt];
        acc[nt] = SWAPPED ? Mma<T>::mma(b.f[kf], a[0].f[kf][nt], c) : Mma<T>::mma(a[0].f[kf][nt], b.f[kf], c);
      }
      b.f[kf] = *reinterpret_cast<const typename Mma<T>::Frag*>(next + kf * KC);
      part(kf);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // All row tiles (RT > 0) of one item.  The epilogue of a row tile has PARTS parts; epi(part, r, acc) is called for parts 0 .. NKF - 1, beside the next one's
  // MFMAs; before_last() is called in front of the last one's, where the weights' registers are free.
  template <bool SWAPPED, int PARTS, typename Epi, typename Before>
  __device__ __forceinline__ void row_steps(const T* Xs, int ldx, int RT, const f32x4 (&start)[NT], Epi epi, Before before_last) const {
    static_assert(PARTS <= NKF, "parts of an epilogue past the last k-fragment would never run");
    const int lane = opaque_tid() & 63;
    const T* next = Xs + (lane & 15) * ldx + lane_piece(lane);
    f32x4 acc0[NT], acc1[NT];
    BRow<T, NKF> b;
#pragma unroll
    for (int kf = 0; kf < NKF; ++kf) b.f[kf] = *reinterpret_cast<const typename Mma<T>::Frag*>(next + kf * KC);
    const auto advance = [&](int r) { next += r + 1 < RT ? 16 * ldx : 0; };
    advance(0);
    row_step<SWAPPED>(acc0, start, b, next, [](int) {});
    int r = 1;
    for (; r + 1 < RT; r += 2) {
      advance(r);
      row_step<SWAPPED>(acc1, start, b, next, [&](int k) { epi(k, r - 1, acc0); });
      advance(r + 1);
      row_step<SWAPPED>(acc0, start, b, next, [&](int k) { epi(k, r, acc1); });
    }
    if (r < RT) {
      row_step<SWAPPED>(acc1, start, b, next, [&](int k) { epi(k, r - 1, acc0); });
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc0[nt] = acc1[nt];
      ++r;
    }
    before_last();
#pragma unroll
    for (int k = 0; k < NKF; ++k) epi(k, r - 1, acc0);
  }
  // run() of a phase of one item per wavefront, over all row tiles.  prefetch_rest() has fetched the bias.
  template <bool SWAPPED, int PARTS, typename Epi>
  __device__ __forceinline__ void run_rows(const T* Xs, int ldx, int RT, Epi epi) const {
    static_assert(KSPLIT == 1 && RSPLIT == 1 && IPW == 1 && N_ITEMS == NW, "one item per wavefront");
    f32x4 b4[NT];
    start_bias(b4, bias0, SWAPPED);
    row_steps<SWAPPED, PARTS>(Xs, ldx, RT, b4, epi, []() {});
  }

  // The same with the bias fetched here and before_last_epi() called between the last MFMAs and the last epilogue: what it requests
  // travels while the epilogue computes.
  template <int PARTS, typename Epi, typename Before>
  __device__ __forceinline__ void run_before(const T* Xs, int ldx, int RT, const float* __restrict__ bias, Epi epi, Before before_last_epi) const {
    static_assert(KSPLIT == 1 && RSPLIT == 1 && IPW == 1, "one item per wavefront");
    if (N_ITEMS >= NW || wave < N_ITEMS) {
      Bias bl;
      load_bias(bl, bias, wave, false);
      row_steps<false, PARTS>(Xs, ldx, RT, bl.v, [&](int k, int r, f32x4 (&acc)[NT]) { epi(k, wave * 16 * NT, r, acc); }, before_last_epi);
    } else {
      before_last_epi();
    }
  }

  // One item per wavefront: row tiles rt0 .. rt0 + HC - 1 unrolled, all accumulators returned
  // (the LayerNorm phases need a row's values in registers across a workgroup barrier).  k-fragment by k-fragment over all row
  // tiles, so that with KSPLIT > 1 the next slice of K is requested into a fragment's registers as soon as that is used; the activations
  // are read kKeepRing fragments ahead.  (In fixed order, see row_step().)
  template <int HC>
  __device__ __forceinline__ void run_keep(const T* Xs, int ldx, int rt0, const f32x4 (&b4)[NT], f32x4 (&acc)[NT][RH]) {
    static_assert(IPW == 1 && HC <= RH, "one item per wavefront");
    typedef typename Mma<T>::Frag Frag;
    constexpr int ALL = NKF_ALL * HC, RING = ALL < kKeepRing ? ALL : kKeepRing;       // activation fragments, k by k and row tile by row tile
    const unsigned lane = opaque_tid() & 63;
    const T* xp = Xs + (16 * rt0 + (lane & 15)) * ldx + lane_piece(lane);
    const Frag* wp = reinterpret_cast<const Frag*>(Wp) + (size_t)((wave % N_OG) * NT) * NKF_ALL * 64;
    const auto read = [&](int f) { return *reinterpret_cast<const Frag*>(xp + 16 * (f % HC) * ldx + f / HC * KC); };
    Frag b[RING];
#pragma unroll
    for (int f = 0; f < RING; ++f) b[f] = read(f);
#pragma unroll
    for (int f = 0; f < ALL; ++f) {
      const int kf = f / HC, r = f % HC;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt][r] = Mma<T>::mma(a[0].f[kf % NKF][nt], b[f % RING], kf == 0 ? b4[nt] : acc[nt][r]);
      if (f + RING < ALL) b[f % RING] = read(f + RING);
      if (r == HC - 1 && kf + NKF < NKF_ALL) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) a[0].f[kf % NKF][nt] = (wp + (nt * NKF_ALL + kf + NKF) * 64)[lane];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = HC; r < RH; ++r) opaque_def(acc[nt][r]);
  }
};

// Reductions over the four lanes m, m + 16, m + 32, m + 48 (one accumulator column) with the gfx950 lane-swap instructions, no LDS round trip:
// permlane32_swap(a, b) returns a's halves and b's as (a.lo, b.lo) and (a.hi, b.hi): a's sums over lanes l, l + 32 in the lower half,
// b's in the upper one; permlane16_swap(a, b) the even and the odd 16-lane rows: (a0, b0, a2, b2) and (a1, b1, a3, b3).
__device__ __forceinline__ float merge32(float a, float b) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float merge16(float a, float b) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
// (the maxima are taken by the instruction itself: fmaxf() on values that come out of a lane swap as plain bits
// is compiled with an extra quieting operation per operand)
__device__ __forceinline__ float raw_max(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Reduction of N = 1, 2 or 4 values over the four lanes of a column (m, m + 16, m + 32, m + 48), `fin` applied, in every lane.  Several
// values share the lane swaps (merge32(), merge16() above): three swaps for two or for four values, where one at a time takes two each.
// Lanes are added as (0 + 2) + (1 + 3) whatever N is, so that a head's result does not depend on the heads that it shares an item with.
template <int N, typename Op, typename Fin>
__device__ __forceinline__ void col_reduce(float (&v)[N], Op op, Fin fin) {
  const auto swap32 = [](float a, float b) { return __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false); };
  const auto swap16 = [](float a, float b) { return __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false); };
  const auto fold = [&](auto p) { return op(__uint_as_float(p[0]), __uint_as_float(p[1])); };
  static_assert(N == 1 || N == 2 || N == 4, "");
  // halves of a: values 0, 1 (N = 1: 0 in both), their lanes 0 + 2 in the even 16-lane rows, 1 + 3 in the odd ones; of b: values 2, 3
  const float a = fold(swap32(v[0], v[N > 1 ? 1 : 0])), b = N == 4 ? fold(swap32(v[N / 2], v[N - 1])) : a;
  const float r = fin(fold(swap16(a, b)));                         // 16-lane rows: values 0, 2, 1, 3 (N = 2: 0, 0, 1, 1)
  if constexpr (N == 1) {
    v[0] = r;
  } else if constexpr (N == 2) {
    const auto p = swap32(r, r);
    v[0] = __uint_as_float(p[0]); v[1] = __uint_as_float(p[1]);
  } else {
    const auto p = swap16(r, r);
    const auto c = swap32(__uint_as_float(p[0]), __uint_as_float(p[0])), d = swap32(__uint_as_float(p[1]), __uint_as_float(p[1]));
    v[0] = __uint_as_float(c[0]); v[1] = __uint_as_float(c[1]);
    v[2] = __uint_as_float(d[0]); v[N - 1] = __uint_as_float(d[1]);
  }
}

// erf-GELU of fp32 features, x * Phi(x) = 0.5 x (1 + erf(x / sqrt 2)), with erf(z) = 1 - 1 / p(z)^16 from
// Abramowitz & Stegun 7.1.28 (six coefficients, |error| <= 3e-7).
// 0.5 x + 0.5 |x| erf(|x|/sqrt 2) = max(x, 0) - |x| / (2 p^16); the polynomial is taken in
// a = |x| directly, q(a) = 2^(1/16) p(a / sqrt 2), so that q^16 = 2 p^16.
constexpr double gelu_coef(double c, int deg) {
  double r = c;
  for (int i = 0; i < deg; ++i) r *= 0.70710678118654752440;              // (1 / sqrt 2)^deg
  double root = 2.0;                                                        // 2^(1 / 16)
  for (int i = 0; i < 4; ++i) {                                             // Newton square roots, constexpr-friendly
    double y = root > 1.0 ? root : 1.0;
    for (int k = 0; k < 60; ++k) y = 0.5 * (y + root / y);
    root = y;
  }
  return r * root;
}
__device__ __forceinline__ float gelu_erf_fast(float x) {
  constexpr float k0 = (float)gelu_coef(1.0, 0), k1 = (float)gelu_coef(0.0705230784, 1),
                  k2 = (float)gelu_coef(0.0422820123, 2), k3 = (float)gelu_coef(0.0092705272, 3),
                  k4 = (float)gelu_coef(0.0001520143, 4), k5 = (float)gelu_coef(0.0002765672, 5),
                  k6 = (float)gelu_coef(0.0000430638, 6);
  const float a = fabsf(x);
  float q = fmaf(k6, a, k5);
  q = fmaf(q, a, k4);
  q = fmaf(q, a, k3);
  q = fmaf(q, a, k2);
  q = fmaf(q, a, k1);
  q = fmaf(q, a, k0);
  q = q * q; q = q * q; q = q * q; q = q * q;
  return fmaf(-a, __builtin_amdgcn_rcpf(q), fmaxf(x, 0.f));
}
// v += swizzled rows of Xs (LDS, pitch ldx), for values in accumulator layout: features o0 .. o0 + 16*NT - 1 of rows 16*(rt0 + r) + m, r < cnt.
template <typename T, int NT, int RH>
__device__ __forceinline__ void add_rows(f32x4 (&v)[NT][RH], const T* Xs, int ldx, int rt0, int cnt, int o0) {
  typedef typename Mma<T>::Vec4 Vec4;
  const int lane = opaque_tid() & 63, m = lane & 15, g = lane >> 4;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < RH; ++r)
      if (r < cnt) {
        const Vec4 xr = *reinterpret_cast<const Vec4*>(Xs + (16 * (rt0 + r) + m) * ldx + o0 + 16 * nt + (4 * g ^ swizzle<T>(m)));
        v[nt][r] += f32x4{to_f32<T>(xr[0]), to_f32<T>(xr[1]), to_f32<T>(xr[2]), to_f32<T>(xr[3])};
      }
}

// (One lane-swap reduction serves two sums of two row tiles, and a row's sums lie together, three 16-byte reads at C = 192
// where twelve 4-byte ones were.  A reduction per sum and 4-byte reads -> this, one session: pass of 3,001 pillars 149.2 -> 147.1 us,
// 30,000 376.7 -> 372.0, 120,000 voxels 682.5 -> 676.4, skewed batch 7,682 -> 7,610.)
// LayerNorm over the C features of every row, for values spread over the workgroup in
// accumulator layout: this wavefront holds features o0 .. o0 + 16*NT - 1 (group og of
// SG = C / (16*NT)) of rows 16*(rt0 + r) + m, r < cnt (cnt = 0: only the barrier).  Per-group sums of x and x^2 (fp32) are
// exchanged through LDS; variance = E[x^2] - mean^2.  Every thread of the workgroup must call it.
// affine(nt, gamma, beta): this lane's four of each for output tile nt; called behind the exchange's barrier, so that they may
// come from LDS that was written before it.
// put(r, row, y): a normalised row's features o0 + 16*nt + 4*g .. + 3, row tile by row tile, every lane of the wavefront together.
template <typename T, int NT, int C, int RH, typename Affine, typename Put>
__device__ __forceinline__ void layer_norm_tile(f32x4 (&v)[NT][RH], int o0, int og, int rt0, int cnt, float* stat,
                                                Affine affine, float eps, Put put) {
  constexpr int SG = C / (16 * NT);
  static_assert(SG * 16 * NT == C && SG <= kStatGroupsMax && SG % 2 == 0, "LayerNorm feature groups");
  const int lane = opaque_tid() & 63, m = lane & 15, g = lane >> 4;
#pragma unroll
  for (int r = 0; r < RH; r += 2) {
    if (r < cnt) {
      float s[2] = {0.f, 0.f}, q[2] = {0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (r + k < RH && r + k < cnt) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) { s[k] += v[nt][r + k][i]; q[k] = fmaf(v[nt][r + k][i], v[nt][r + k][i], q[k]); }
        }
      // the sums over the four lanes of a column, of two row tiles at once: lane group g ends up with quantity g >> 1 of row tile r + (g & 1)
      const float sum = merge16(merge32(s[0], q[0]), merge32(s[1], q[1]));
      if ((g & 1) == 0 || (r + 1 < RH && r + 1 < cnt)) stat[((16 * (rt0 + r + (g & 1)) + m) * SG + og) * 2 + (g >> 1)] = sum;
    }
  }
  lds_barrier();
  f32x4 ga[NT], be[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) affine(nt, ga[nt], be[nt]);
#pragma unroll
  for (int r = 0; r < RH; ++r) {
    if (r < cnt) {
      const int row = 16 * (rt0 + r) + m;
      float s = 0.f, q = 0.f;
#pragma unroll
      for (int k = 0; k < SG / 2; ++k) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(stat + (row * SG + 2 * k) * 2);
        s += t[0]; q += t[1]; s += t[2]; q += t[3];
      }
      const float mean = s * (1.0f / C);
      const float rs = __builtin_amdgcn_rsqf(fmaxf(fmaf(-mean, mean, q * (1.0f / C)), 0.f) + eps);
      const float sh = -mean * rs;
      f32x4 y[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[nt][i] = fmaf(fmaf(v[nt][r][i], rs, sh), ga[nt][i], be[nt][i]);
      put(r, row, y);
    }
  }
}

// dst fragment order <- src [out, in]; one thread per 16-byte lane slot.
template <typename T>
__global__ void k_pack(const T* __restrict__ src, T* __restrict__ dst, int out, int k) {
  constexpr int KC = Mma<T>::KC, KL = Mma<T>::KL;
  const int nkf = k / KC;
  const long long slot = (long long)blockIdx.x * blockDim.x + threadIdx.x;     // (tile, kf, lane)
  if (slot >= (long long)(out / 16) * nkf * 64) return;
  const int lane = (int)(slot & 63), kf = (int)((slot >> 6) % nkf), tile = (int)((slot >> 6) / nkf);
  const T* s = src + (size_t)(tile * 16 + (lane & 15)) * k + kf * KC + (lane >> 4) * KL;
  T* d = dst + (size_t)slot * KL;
#pragma unroll
  for (int e = 0; e < KL; ++e) d[e] = s[e];
}

