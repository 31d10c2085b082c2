// dsvt_vfe: the step before the first DSVT block (Sec. 3.1 overview: the point cloud becomes sparse voxels
// through a voxel feature encoding module; the paper cites earlier pillar encoders for it).  Built here: an
// optional per-point linear map followed by the channel-wise maximum over each voxel's points.
//
// Voxels are found without a sort: the points are counted in a map over the grid's cells, in key order, and a scan
// over its words of 32 cells numbers the non-empty ones in ascending key and gives every voxel a run of rows; the value
// a point's atomic returned is its place there (a counting sort), and wavefronts with equal shares of the rows take
// the maxima from LDS.  (Grids large for their points: the map holds a byte per cell, and the points are counted by voxel once
// the voxels are numbered.  See prefer_by_cell.)  The order of a voxel's points in its
// run varies from call to call, the maximum does not.  Bound by the launches and by the latency of the
// atomics and loads inside them, not by bytes: points are read twice and copied once, the feature rows written once.
#include "common.h"
#include "block_scan.h"

#include <hip/hip_bf16.h>

namespace {

constexpr int kMaxFin = 16;
constexpr uint32_t kOutside = 0xFFFFFFFFu;

struct VfeGeom {
  int32_t grid[3], batch, f_in;
  float lo[3], sz[3];
};

// Cell key ((b*X + x)*Y + y)*Z + z of a point, or kOutside.  The cell is decided in float32, one rounded
// operation at a time (no fused multiply-add, no reciprocal): t = (p - lo) / size, inside iff 0 <= t < cells.
__device__ __forceinline__ uint32_t point_key(const VfeGeom& g, const float* __restrict__ p, int32_t b, int4* cell) {
  if (b < 0 || b >= g.batch) return kOutside;
  int32_t c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float t = __fdiv_rn(__fsub_rn(p[a], g.lo[a]), g.sz[a]);
    if (!(t >= 0.f && t < (float)g.grid[a])) return kOutside;     // NaN fails both
    c[a] = (int32_t)t;
  }
  if (cell) *cell = make_int4(b, c[0], c[1], c[2]);
  return (uint32_t)(((b * g.grid[0] + c[0]) * g.grid[1] + c[1]) * g.grid[2] + c[2]);
}

// 16 bytes of the cell map per thread, and the per-voxel point counts.
__global__ void kv_clear(uint4* __restrict__ cell_map, int64_t n16, int32_t* __restrict__ count, int64_t n_count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n16) cell_map[i] = make_uint4(0u, 0u, 0u, 0u);
  if (i < n_count) count[i] = 0;
}

// Occupancy goes into a byte per cell with a plain store: every writer stores the same 1, so no atomic is needed.
// (Atomic ORs into a bitmap queue up on the few cache lines next to the sensor, where a pillar collects a hundred
// points and a line holds a thousand cells: 28 us for 180,000 points against 8 us this way.)
__global__ void kv_mark(VfeGeom g, const float* __restrict__ points, const int32_t* __restrict__ point_batch, int32_t n,
                        uint8_t* __restrict__ cell_map, uint32_t* __restrict__ keys) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t key = point_key(g, points + (int64_t)i * g.f_in, point_batch ? point_batch[i] : 0, nullptr);
  keys[i] = key;
  if (key != kOutside) cell_map[key] = 1;
}

// 32 cells' bytes (each 0 or 1) -> one bitmap word, bit k = cell 32 w + k.
__global__ void kv_pack(const uint4* __restrict__ cell_map, int64_t n_words, uint32_t* __restrict__ bitmap) {
  const int64_t wd = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (wd >= n_words) return;
  const uint4 a = cell_map[2 * wd], b = cell_map[2 * wd + 1];
  const uint32_t q[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t word = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) word |= ((q[k] * 0x01020408u) >> 24) << (4 * k);     // the four low bits of four bytes
  bitmap[wd] = word;
}

// Voxel index of every point (rank of its cell among the occupied ones) and its place among the voxel's points.
__global__ void kv_count(const uint32_t* __restrict__ keys, int32_t n, const uint32_t* __restrict__ bitmap,
                         const int32_t* __restrict__ word_prefix, int32_t max_voxels, int32_t* __restrict__ count,
                         int32_t* __restrict__ point_vox, int32_t* __restrict__ point_pos, int32_t* __restrict__ status) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t key = keys[i];
  int32_t v = -1, pos = 0;
  if (key != kOutside) {
    const uint32_t word = key >> 5, bit = key & 31u;
    v = word_prefix[word] + __popc(bitmap[word] & ((1u << bit) - 1u));
    if (v >= max_voxels) { atomicOr(status, DSVT_ST_VOXEL_OVERFLOW); v = -1; }
    else pos = atomicAdd(&count[v], 1);
  }
  point_vox[i] = v;
  point_pos[i] = pos;
}

// Points counted by cell instead (see prefer_by_cell): a counter per cell takes the marks, and the value a point's atomic
// returns is its place among the voxel's points, so that neither kv_count nor a scan of the voxels' counts is needed.
__global__ void kv_mark_count(VfeGeom g, const float* __restrict__ points, const int32_t* __restrict__ point_batch, int32_t n,
                              uint32_t* __restrict__ cell_cnt, uint32_t* __restrict__ keys, int32_t* __restrict__ point_pos) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t key = point_key(g, points + (int64_t)i * g.f_in, point_batch ? point_batch[i] : 0, nullptr);
  keys[i] = key;
  if (key != kOutside) point_pos[i] = (int32_t)atomicAdd(&cell_cnt[key], 1u);
}

// A thread per cell, 32 cells a bitmap word: the word, how many of its cells are occupied and how many points they hold,
// and in the place of each cell's counter -- where the word has an occupied one, no other is looked at again -- the points
// of the word's cells before it.
__global__ void kv_pack_count(uint32_t* __restrict__ cell_cnt, int64_t n_words, uint32_t* __restrict__ bitmap,
                              uint32_t* __restrict__ word_vox, uint32_t* __restrict__ word_rows) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;      // (whole wavefronts: n_words is a multiple of 64)
  if (i >= n_words * 32) return;
  const int32_t lane = threadIdx.x & 63;
  const uint32_t c = cell_cnt[i];
  const uint64_t occ = __ballot(c != 0u);
  uint32_t incl = c;
#pragma unroll
  for (int32_t d = 1; d < 32; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, 32);
    if ((lane & 31) >= d) incl += up;
  }
  const uint32_t word = (uint32_t)(occ >> (lane & 32));
  if (word != 0u) cell_cnt[i] = incl - c;
  if ((lane & 31) == 31) {
    bitmap[i >> 5] = word;
    word_vox[i >> 5] = (uint32_t)__popc(word);
    word_rows[i >> 5] = incl;
  }
}

// Where kv_place finds a point's voxel and run: by voxel (kv_count's arrays), or by cell.
struct PlaceSrc {
  const int32_t *point_vox, *offs;                                    // by voxel
  const uint32_t *keys, *bitmap, *cell_before;                        // by cell
  const int32_t *vox_prefix, *row_prefix;
  int32_t max_voxels;
  int32_t *n_rows, *status;
};

// Counting sort, second half: every point's row copied to its voxel's run, so that the reduction reads
// consecutive (zero-padded) rows; run_info[j] = (voxel of row j, first row of its run, first row of the next run).
// The first point of a voxel also writes the voxel's coordinates.
template <int PITCH4, bool BY_CELL>
__global__ void kv_place(VfeGeom g, const float* __restrict__ points, const int32_t* __restrict__ point_batch,
                         PlaceSrc s, const int32_t* __restrict__ point_pos, int32_t n, float4* __restrict__ sorted,
                         int4* __restrict__ run_info, int32_t* __restrict__ coords) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int32_t v, start, end;
  if constexpr (BY_CELL) {
    const uint32_t key = s.keys[i];
    if (key == kOutside) return;
    const uint32_t word = key >> 5, bit = key & 31u;
    v = s.vox_prefix[word] + __popc(s.bitmap[word] & ((1u << bit) - 1u));
    if (v >= s.max_voxels) { atomicOr(s.status, DSVT_ST_VOXEL_OVERFLOW); return; }
    start = s.row_prefix[word] + (int32_t)s.cell_before[key];
    end = bit == 31u ? s.row_prefix[word + 1] : s.row_prefix[word] + (int32_t)s.cell_before[key + 1];
  } else {
    v = s.point_vox[i];
    if (v < 0) return;
    start = s.offs[v];
    end = s.offs[v + 1];
  }
  const int32_t pos = point_pos[i], f_in = g.f_in;
  const int32_t j = start + pos;                             // j < end <= n
  const float* src = points + (int64_t)i * f_in;
  float f[4 * PITCH4];                                       // rows padded with zeros to whole 16-byte pieces
#pragma unroll
  for (int k = 0; k < 4 * PITCH4; ++k) f[k] = k < f_in ? src[k] : 0.f;
#pragma unroll
  for (int k4 = 0; k4 < PITCH4; ++k4)
    sorted[(int64_t)j * PITCH4 + k4] = make_float4(f[4 * k4], f[4 * k4 + 1], f[4 * k4 + 2], f[4 * k4 + 3]);
  run_info[j] = make_int4(v, start, end, 0);
  if (pos == 0) {
    int4 cell = make_int4(0, 0, 0, 0);
    point_key(g, src, point_batch ? point_batch[i] : 0, &cell);
    reinterpret_cast<int4*>(coords)[v] = cell;
    if (BY_CELL && v == s.max_voxels - 1) *s.n_rows = end;   // the rows of the voxels that are kept (nobody reads it here)
  }
}

// Work is split by points, not by voxels (a pillar next to the sensor holds a hundred points, most hold one): a
// wavefront takes the voxels whose runs start inside its kQuota rows of the sorted array; what it needs to know
// about them comes from run_info at its first row and at the next workgroup's, so that its first loads do not
// wait for one another.  A wavefront works alone; lane l owns channels l, l + 64, ... and keeps their rows of
// w in registers, so a row fetched from LDS serves all of them.
// The rows are staged in LDS (kStage of them; a run that reaches further is read from memory), then every thread
// walks them voxel by voxel -- all lanes read the same row, so an LDS read is one broadcast -- and writes the
// voxel's maximum when its run ends.  h = b[c] + sum_k w[c,k] f[k] in k order; w == NULL: h = f[c].
// Bound by the latency of its loads, so as few of them as possible wait for one another: the weights and the (uniform)
// run_info entries first, then the rows and their run_info together; run ends go from lane to lane in a register and
// no wavefront waits for another.  180,000 points, C = 192: 19.6 -> 16.4 us under the profiler, the whole call 54.0 ->
// 51.7 (quotas of 8 and 32 rows: 52.3 and 49.9 where 16 takes 49.2 and 49.5).
constexpr int kQuota = 16, kStage = 128, kRedWaves = 4;
static_assert(kQuota <= 64 && (kQuota & (kQuota - 1)) == 0, "a run starts in the first row of some lane");

template <int FIN, int CPL>
__device__ __forceinline__ void fold_row(const float4* __restrict__ row, const float (&wr)[CPL][FIN], const float (&b0)[CPL],
                                         float (&best)[CPL]) {
  constexpr int P4 = (FIN + 3) / 4;
  float f[4 * P4];
#pragma unroll
  for (int k4 = 0; k4 < P4; ++k4) {
    const float4 t = row[k4];
    f[4 * k4] = t.x; f[4 * k4 + 1] = t.y; f[4 * k4 + 2] = t.z; f[4 * k4 + 3] = t.w;
  }
#pragma unroll
  for (int m = 0; m < CPL; ++m) {
    float h = b0[m];
#pragma unroll
    for (int k = 0; k < FIN; ++k) h = fmaf(wr[m][k], f[k], h);
    best[m] = fmaxf(best[m], h);
  }
}

// What a wavefront stored to LDS is what its later reads see: its LDS operations run in order, so only the compiler has
// to keep them so.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// FIN: the point row's length rounded up to a supported one (the extra columns of w are zero); the rows' pitch is
// ceil(FIN / 4) 16-byte pieces.  CPL: channels per lane.
template <int FIN, int CPL>
__global__ void __launch_bounds__(64 * kRedWaves) kv_reduce(const float4* __restrict__ sorted, const int4* __restrict__ run_info,
                                                const int32_t* __restrict__ n_rows_dev, const int32_t* __restrict__ n_voxels,
                                                int32_t max_voxels, int32_t n_points, int32_t f_in,
                                                const float* __restrict__ w, const float* __restrict__ bias,
                                                int32_t relu, int32_t C, int32_t bf16_out, void* __restrict__ x) {
  constexpr int PITCH4 = (FIN + 3) / 4, PITCH = 4 * PITCH4;
  // Every wavefront works on a quota of its own and shares nothing with the others: four of them form a
  // workgroup only so that the dispatcher spreads them over a compute unit's four SIMDs (as one-wavefront
  // workgroups they were packed onto a third of the chip).
  __shared__ float4 rows_all[kRedWaves][kStage * PITCH4];
  __shared__ int32_t end_all[kRedWaves][kQuota + 1];    // last row + 1 of each of the wavefront's voxels, relative; one not used
  const int32_t lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x >> 6);
  float4* rows_s = rows_all[wv];
  int32_t* end_s = end_all[wv];
  const int32_t part = blockIdx.x * kRedWaves + wv;
  // The weights are on their way before the first wait.  Every lane loads some element, so that no branch (and no wait)
  // comes between the loads; without w or bias, or past the last channel, it is one that is not used.
  const float* any = reinterpret_cast<const float*>(run_info);
  const float *wp = w ? w : any, *bp = bias ? bias : any;
  float wr[CPL][FIN], b0[CPL];
#pragma unroll
  for (int m = 0; m < CPL; ++m) {
    const int32_t c = lane + 64 * m;
#pragma unroll
    for (int k = 0; k < FIN; ++k) {
      const bool in = w && c < C && k < f_in;
      const float t = wp[in ? c * f_in + k : 0];
      wr[m][k] = in ? t : 0.f;
    }
    const bool in = bias && c < C;
    const float t = bp[in ? c : 0];
    b0[m] = in ? t : 0.f;
  }
  // The first voxel whose run starts at or after the wavefront's first row, and that row; the same for the next wavefront's.
  // (Uniform: scalar loads.)
  const int32_t total = *n_rows_dev, nv = min(*n_voxels, max_voxels), j0 = part * kQuota, j1 = j0 + kQuota;
  const int4 at0 = run_info[min(j0, n_points - 1)], at1 = run_info[min(j1, n_points - 1)];
  auto voxel_at = [&](int32_t j, int4 at) { return j >= total ? nv : at.y == j ? at.x : at.x + 1; };   // (beyond row `total`
  auto row_at = [&](int32_t j, int4 at) { return j >= total ? total : at.y == j ? j : at.z; };         // `at` means nothing)
  const int32_t va = voxel_at(j0, at0), n_vox = voxel_at(j1, at1) - va;      // n_vox <= kQuota: every run has a row; <= 0:
  const int32_t p_begin = row_at(j0, at0), n_own = n_vox > 0 ? row_at(j1, at1) - p_begin : 0;      // nothing to do
  if (lane < n_own) {                                     // the runs start in the first kQuota rows
    const int4 info = run_info[p_begin + lane];
    float4 row[PITCH4];
#pragma unroll
    for (int k4 = 0; k4 < PITCH4; ++k4) row[k4] = sorted[(int64_t)(p_begin + lane) * PITCH4 + k4];
    end_s[info.y == p_begin + lane ? info.x - va : kQuota] = info.z - p_begin;   // a run's first row announces its end
#pragma unroll
    for (int k4 = 0; k4 < PITCH4; ++k4) rows_s[lane * PITCH4 + k4] = row[k4];
  }
  for (int32_t r = lane + 64; r < min(n_own, (int32_t)kStage); r += 64) {
#pragma unroll
    for (int k4 = 0; k4 < PITCH4; ++k4) rows_s[r * PITCH4 + k4] = sorted[(int64_t)(p_begin + r) * PITCH4 + k4];
  }
  wave_lds_order();
  const int32_t ends = end_s[lane & (kQuota - 1)];             // (entries past the last voxel's are not used)
  const float* rows_f = reinterpret_cast<const float*>(rows_s);
  const float* sorted_f = reinterpret_cast<const float*>(sorted);
  int32_t lo = 0;
  for (int32_t vl = 0; vl < n_vox; ++vl) {
    const int32_t hi = __builtin_amdgcn_readlane(ends, vl), hi_s = min(hi, (int32_t)kStage);
    float best[CPL];
#pragma unroll
    for (int m = 0; m < CPL; ++m) best[m] = -INFINITY;
    if (w) {
#pragma unroll 2
      for (int32_t q = lo; q < hi_s; ++q) fold_row<FIN, CPL>(rows_s + q * PITCH4, wr, b0, best);
      for (int32_t q = max(lo, (int32_t)kStage); q < hi; ++q)             // the part of a long run that was not staged
        fold_row<FIN, CPL>(sorted + (int64_t)(p_begin + q) * PITCH4, wr, b0, best);
    } else if (lane < C) {                                // no linear map (C = f_in <= 16): channel `lane` of the row
      for (int32_t q = lo; q < hi_s; ++q) best[0] = fmaxf(best[0], rows_f[q * PITCH + lane] + b0[0]);
      for (int32_t q = max(lo, (int32_t)kStage); q < hi; ++q)
        best[0] = fmaxf(best[0], sorted_f[(int64_t)(p_begin + q) * PITCH + lane] + b0[0]);
    }
#pragma unroll
    for (int m = 0; m < CPL; ++m) {
      const int32_t c = lane + 64 * m;
      const float y = relu ? fmaxf(best[m], 0.f) : best[m];
      if (c < C) {
        if (bf16_out) reinterpret_cast<__hip_bfloat16*>(x)[(int64_t)(va + vl) * C + c] = __float2bfloat16(y);
        else reinterpret_cast<float*>(x)[(int64_t)(va + vl) * C + c] = y;
      }
    }
    lo = hi;
  }
}

struct VfePlan {
  VfeGeom g;
  int64_t n_words;
  size_t off_cells, off_bitmap, off_prefix, off_count, off_offs, off_keys, off_vox, off_pos, off_info, off_nrows, off_sorted, total;
  // the layout of a call that counts points by cell; row prefixes lie words_pitch behind the voxel prefixes, likewise the counts
  int64_t cells, words_pitch;
  size_t off_cnt2, off_bitmap2, off_words2, off_prefix2, off_keys2, off_pos2, off_info2, off_nrows2, off_sorted2, total2;
};

int make_plan(const dsvt_vfe_cfg* cfg, int32_t n_points, int32_t max_voxels, VfePlan* pl) {
  if (!cfg || n_points <= 0 || max_voxels <= 0 || cfg->batch <= 0) return DSVT_EINVAL;
  if (cfg->f_in < 3 || cfg->f_in > kMaxFin || cfg->C <= 0 || cfg->C > 512) return DSVT_EINVAL;
  if (cfg->dtype != DSVT_F32 && cfg->dtype != DSVT_BF16) return DSVT_EINVAL;
  if (!cfg->w && cfg->C != cfg->f_in) return DSVT_EINVAL;
  int64_t cells = cfg->batch;
  for (int a = 0; a < 3; ++a) {
    if (cfg->grid[a] <= 0 || !(cfg->voxel_size[a] > 0.f) || !(cfg->range_min[a] == cfg->range_min[a])) return DSVT_EINVAL;
    cells *= cfg->grid[a];
    pl->g.grid[a] = cfg->grid[a];
    pl->g.lo[a] = cfg->range_min[a];
    pl->g.sz[a] = cfg->voxel_size[a];
  }
  if (cells >= (1ll << 31)) return DSVT_EUNSUPPORTED;
  if ((int64_t)max_voxels * cfg->C >= (1ll << 39)) return DSVT_EINVAL;
  pl->g.batch = cfg->batch;
  pl->g.f_in = cfg->f_in;
  pl->n_words = (int64_t)dsvt_align_up((size_t)dsvt_ceil_div(cells, 32), 64);
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off = dsvt_align_up(off + bytes, 256); return o; };
  pl->off_cells = take((size_t)pl->n_words * 32);
  pl->off_bitmap = take((size_t)pl->n_words * 4);
  pl->off_prefix = take((size_t)pl->n_words * 4);
  pl->off_count = take(((size_t)max_voxels + 1) * 4);
  pl->off_offs = take(((size_t)max_voxels + 1) * 4);
  pl->off_keys = take((size_t)n_points * 4);
  pl->off_vox = take((size_t)n_points * 4);
  pl->off_pos = take((size_t)n_points * 4);
  pl->off_info = take((size_t)n_points * 16);
  pl->off_nrows = take(4);
  pl->off_sorted = take((size_t)n_points * ((cfg->f_in + 3) / 4) * 16);
  pl->total = off;
  pl->cells = cells;
  pl->words_pitch = pl->n_words + 64;                            // room for the entry behind the last word's
  off = 0;
  pl->off_cnt2 = take((size_t)pl->n_words * 32 * 4);
  pl->off_bitmap2 = take((size_t)pl->n_words * 4);
  pl->off_words2 = take((size_t)pl->words_pitch * 8);
  pl->off_prefix2 = take((size_t)pl->words_pitch * 8);
  pl->off_keys2 = take((size_t)n_points * 4);
  pl->off_pos2 = take((size_t)n_points * 4);
  pl->off_info2 = take((size_t)n_points * 16);
  pl->off_nrows2 = take(4);
  pl->off_sorted2 = take((size_t)n_points * ((cfg->f_in + 3) / 4) * 16);
  pl->total2 = off;
  return DSVT_OK;
}

// Whether a call counts its points by cell: six launches in a row where counting by voxel takes eight, for 4 bytes a cell
// cleared, added up and scanned instead of one -- worth it on small grids whatever the points, on larger ones for many points
// only.  By voxel -> by cell, us, 468 x 468 cells a layer, C = 192, 5,000 / 20,000 / 60,000 / 130,000 points: 1 layer 28 -> 24,
// 30 -> 25, 37 -> 31, 42 -> 41; 6 layers (1.3 M cells) 31 -> 30, 34 -> 32, 42 -> 39, 56 -> 50; 8 layers 32 -> 32, 35.5 -> 34.6, 45 ->
// 43, 58 -> 54; 12 layers 34 -> 37, 38 -> 40, 47.7 -> 47.4, 61 -> 58; 24 layers 42 -> 51, 46 -> 52, 55 -> 57, 69 -> 67; 32 layers
// (7.0 M) 45 -> 55, 50 -> 55, 60 -> 60, 74 -> 71 (400,000 points: 123 -> 118).  At 16 layers the larger frames go either way with
// where the buffers lie (180,000 points 73 -> 70 or 78).  kByCellMax bounds the counters' 32 MB.
constexpr int64_t kByCellMax = 1ll << 23, kByCellAny = 1500000, kByCellPoints = 80000;
bool prefer_by_cell(const VfePlan& pl, int32_t n_points) {
  return pl.cells <= kByCellMax && (n_points >= kByCellPoints || pl.cells <= kByCellAny + 20 * (int64_t)n_points);
}
// A call without the scratch for it counts by voxel.  (What fewer points take is never more than what more points take, so
// scratch for the largest frame serves the others.)
bool count_by_cell(const VfePlan& pl, int32_t n_points, size_t ws_bytes) { return prefer_by_cell(pl, n_points) && pl.total2 <= ws_bytes; }
// Scratch a call asks for: room for the layout it would use, and at least for counting by voxel.
size_t vfe_scratch(const VfePlan& pl, int32_t n_points) { return prefer_by_cell(pl, n_points) && pl.total2 > pl.total ? pl.total2 : pl.total; }

}  // namespace

extern "C" int dsvt_vfe_workspace_size(const dsvt_vfe_cfg* cfg, int32_t n_points, int32_t max_voxels, size_t* bytes) {
  if (!bytes) return DSVT_EINVAL;
  VfePlan pl;
  const int rc = make_plan(cfg, n_points, max_voxels, &pl);
  if (rc != DSVT_OK) return rc;
  *bytes = vfe_scratch(pl, n_points);
  return DSVT_OK;
}

extern "C" int dsvt_vfe(const dsvt_vfe_cfg* cfg, const float* points, const int32_t* point_batch, int32_t n_points,
                        int32_t* coords, void* x, int32_t* n_voxels, int32_t max_voxels, void* ws, size_t ws_bytes,
                        int32_t* status, void* stream) {
  VfePlan pl;
  const int rc = make_plan(cfg, n_points, max_voxels, &pl);
  if (rc != DSVT_OK) return rc;
  if (!points || !coords || !x || !n_voxels || !ws || !status) return DSVT_EINVAL;
  if (cfg->batch > 1 && !point_batch) return DSVT_EINVAL;
  if (((uintptr_t)coords | (uintptr_t)ws) & 15u) return DSVT_EINVAL;
  if (ws_bytes < pl.total) return DSVT_ENOSPC;
  hipStream_t st = (hipStream_t)stream;
  char* base = reinterpret_cast<char*>(ws);
  const bool by_cell = count_by_cell(pl, n_points, ws_bytes);
  uint32_t* bitmap = reinterpret_cast<uint32_t*>(base + (by_cell ? pl.off_bitmap2 : pl.off_bitmap));
  uint32_t* keys = reinterpret_cast<uint32_t*>(base + (by_cell ? pl.off_keys2 : pl.off_keys));
  int32_t* pos = reinterpret_cast<int32_t*>(base + (by_cell ? pl.off_pos2 : pl.off_pos));
  float4* sorted4 = reinterpret_cast<float4*>(base + (by_cell ? pl.off_sorted2 : pl.off_sorted));
  int4* run_info = reinterpret_cast<int4*>(base + (by_cell ? pl.off_info2 : pl.off_info));
  int32_t* n_rows = reinterpret_cast<int32_t*>(base + (by_cell ? pl.off_nrows2 : pl.off_nrows));
  const int tb = 256;
  const unsigned pb = (unsigned)dsvt_ceil_div(n_points, tb);
  {
    dsvt_prof_scope ps(DSVT_K_VFE_GROUP, st);
    PlaceSrc src = {};
    if (by_cell) {
      uint32_t* cnt = reinterpret_cast<uint32_t*>(base + pl.off_cnt2);
      uint32_t* words = reinterpret_cast<uint32_t*>(base + pl.off_words2);
      int32_t* prefix = reinterpret_cast<int32_t*>(base + pl.off_prefix2);
      const int64_t n16 = pl.n_words * 8;
      kv_clear<<<(unsigned)dsvt_ceil_div(n16, tb), tb, 0, st>>>(reinterpret_cast<uint4*>(cnt), n16, nullptr, 0);
      kv_mark_count<<<pb, tb, 0, st>>>(pl.g, points, point_batch, n_points, cnt, keys, pos);
      kv_pack_count<<<(unsigned)dsvt_ceil_div(pl.n_words * 32, tb), tb, 0, st>>>(cnt, pl.n_words, bitmap, words, words + pl.words_pitch);
      k_block_scan<false, true><<<dim3(block_scan_grid(pl.n_words), 2), 1024, 0, st>>>(words, prefix, pl.n_words, nullptr, n_voxels,
                                                                                     pl.words_pitch, n_rows);
      src.keys = keys; src.bitmap = bitmap; src.cell_before = cnt;
      src.vox_prefix = prefix; src.row_prefix = prefix + pl.words_pitch;
      src.max_voxels = max_voxels; src.n_rows = n_rows; src.status = status;
    } else {
      uint8_t* cells = reinterpret_cast<uint8_t*>(base + pl.off_cells);
      int32_t* prefix = reinterpret_cast<int32_t*>(base + pl.off_prefix);
      int32_t* count = reinterpret_cast<int32_t*>(base + pl.off_count);
      int32_t* offs = reinterpret_cast<int32_t*>(base + pl.off_offs);
      int32_t* vox = reinterpret_cast<int32_t*>(base + pl.off_vox);
      const int64_t n_count = (int64_t)max_voxels + 1, n16 = pl.n_words * 2;
      const int64_t n_clear = n16 > n_count ? n16 : n_count;
      kv_clear<<<(unsigned)dsvt_ceil_div(n_clear, tb), tb, 0, st>>>(reinterpret_cast<uint4*>(cells), n16, count, n_count);
      kv_mark<<<pb, tb, 0, st>>>(pl.g, points, point_batch, n_points, cells, keys);
      kv_pack<<<(unsigned)dsvt_ceil_div(pl.n_words, tb), tb, 0, st>>>(reinterpret_cast<const uint4*>(cells), pl.n_words, bitmap);
      k_block_scan<true><<<block_scan_grid(pl.n_words), 1024, 0, st>>>(bitmap, prefix, pl.n_words, nullptr, n_voxels);
      kv_count<<<pb, tb, 0, st>>>(keys, n_points, bitmap, prefix, max_voxels, count, vox, pos, status);
      k_block_scan<false, true><<<block_scan_grid(max_voxels), 1024, 0, st>>>(reinterpret_cast<const uint32_t*>(count), offs, max_voxels, n_voxels, n_rows);
      src.point_vox = vox; src.offs = offs;
    }
#define DSVT_VFE_PLACE(P4)                                                                                                        \
    if (by_cell) kv_place<P4, true><<<pb, tb, 0, st>>>(pl.g, points, point_batch, src, pos, n_points, sorted4, run_info, coords);    \
    else kv_place<P4, false><<<pb, tb, 0, st>>>(pl.g, points, point_batch, src, pos, n_points, sorted4, run_info, coords);           \
    break
    switch ((cfg->f_in + 3) / 4) {
      case 1: DSVT_VFE_PLACE(1);
      case 2: DSVT_VFE_PLACE(2);
      case 3: DSVT_VFE_PLACE(3);
      default: DSVT_VFE_PLACE(4);
    }
#undef DSVT_VFE_PLACE
  }
  {
    dsvt_prof_scope ps(DSVT_K_VFE_REDUCE, st);
    const unsigned rb = (unsigned)dsvt_ceil_div(n_points, kQuota * kRedWaves);
    const int cpl = (cfg->C + 63) / 64;                                        // channels per lane: 1, 2, 3, 4 or 8
    const int fin = cfg->f_in <= 6 ? (cfg->f_in < 4 ? 4 : cfg->f_in) : cfg->f_in <= 8 ? 8 : cfg->f_in <= 12 ? 12 : 16;
#define DSVT_VFE_LAUNCH(FIN, CPL)                                                                                  \
    kv_reduce<FIN, CPL><<<rb, 64 * kRedWaves, 0, st>>>(sorted4, run_info, n_rows, n_voxels, max_voxels, n_points, cfg->f_in,    \
                                           cfg->w, cfg->b, cfg->relu, cfg->C, cfg->dtype == DSVT_BF16, x)
#define DSVT_VFE_CPL(FIN)                                                                                          \
    switch (cpl) {                                                                                                 \
      case 1: DSVT_VFE_LAUNCH(FIN, 1); break;                                                                      \
      case 2: DSVT_VFE_LAUNCH(FIN, 2); break;                                                                      \
      case 3: DSVT_VFE_LAUNCH(FIN, 3); break;                                                                      \
      case 4: DSVT_VFE_LAUNCH(FIN, 4); break;                                                                      \
      default: DSVT_VFE_LAUNCH(FIN, 8); break;                                                                     \
    }
    switch (fin) {
      case 4: DSVT_VFE_CPL(4); break;
      case 5: DSVT_VFE_CPL(5); break;
      case 6: DSVT_VFE_CPL(6); break;
      case 8: DSVT_VFE_CPL(8); break;
      case 12: DSVT_VFE_CPL(12); break;
      default: DSVT_VFE_CPL(16); break;
    }
#undef DSVT_VFE_CPL
#undef DSVT_VFE_LAUNCH
  }
  DSVT_HIP_TRY(hipGetLastError());
  return DSVT_OK;
}
