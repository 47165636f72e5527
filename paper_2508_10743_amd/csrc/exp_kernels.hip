// Scaling and squaring (Section 3, "Diffeomorphisms") and its adjoint.
//
// Forward step: u_{t+1}(x) = u_t(x) + u_t(x + u_t(x)), trilinear with border
// clamping; the first step reads v and scales it by 2^-N on the fly.
//
// Adjoint step: g_t(y) = g(y) + J_t(y)^T g(y) + sum_x sum_k [corner_k(x) = y] w_k(x) g(x)
// with g = g_{t+1}.  The scatter term is computed owner-side, as a gather, so
// that no global atomics and no zero-fill pass are needed and each output value
// is written once: where every cell lies within one voxel, a target sums its 27
// neighbours, weighted by hat functions of their displacements; beyond, a block
// bins the source voxels whose trilinear cells touch its targets by cell (one LDS
// integer atomic per source) and every target sums over the sources binned in
// its 8 neighbouring cells.  Which source voxels to look at follows from the
// offsets (cell index - voxel index) recorded per tile of 32 (d2) x 8 (d1) x 8
// (d0) voxels by the forward step, or before the adjoint for the subjects that
// need them.  (Float atomics in LDS are serialised lane by lane on this hardware:
// scattering the 24 weighted corner values of every source with them costs an
// order of magnitude more than the binning.)
#include <climits>

#include "darc_kernels.hpp"
#include "voxel_bodies.hpp"

namespace darc {

namespace {

constexpr int ETX = 32, ETY = 8, ETZ = 8;
constexpr int ENT = ETX * ETY;             // threads per block

struct TileGeom {
  Geom g;
  int ntx, nty, ntz, ntiles;
  uint32_t total;  // ntiles * subjects
};

TileGeom make_tiles(const Geom& g, int n) {
  TileGeom t;
  t.g = g;
  t.ntx = (g.d2 + ETX - 1) / ETX;
  t.nty = (g.d1 + ETY - 1) / ETY;
  t.ntz = (g.d0 + ETZ - 1) / ETZ;
  t.ntiles = t.ntx * t.nty * t.ntz;
  t.total = static_cast<uint32_t>(t.ntiles) * n;
  return t;
}

// Minimum or maximum over the 64 lanes of a wave (every lane active), by DPP
// lane moves that need no LDS: shifts by 1, 2, 4 and 8 lanes within each
// 16-lane row (a lane with no source lane takes the identity) leave each
// row's extreme in its lane 15; broadcasting lane 15 into the next row and
// lane 31 into rows 2 and 3 folds the four rows into lane 63.
template <bool MAX>
__device__ __forceinline__ int wave_extreme(int x) {
  constexpr int kRowShr = 0x110, kBcast15 = 0x142, kBcast31 = 0x143;
  constexpr int id = MAX ? INT_MIN : INT_MAX;
  auto op = [](int a, int b) { return MAX ? max(a, b) : min(a, b); };
  x = op(x, __builtin_amdgcn_update_dpp(id, x, kRowShr + 1, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(id, x, kRowShr + 2, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(id, x, kRowShr + 4, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(id, x, kRowShr + 8, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(id, x, kBcast15, 0xa, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(id, x, kBcast31, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}
__device__ __forceinline__ int wave_min(int x) { return wave_extreme<false>(x); }
__device__ __forceinline__ int wave_max(int x) { return wave_extreme<true>(x); }

// Per-tile records used by the adjoint: boxes[(s * ntiles + tile) * 8 + {0,1,2}]
// = min over the tile's voxels x of i_d(x) - x_d along d0, d1, d2 (i = cell
// index of x + u(x)), [.. + {3,4,5}] = the max; so the corners a voxel x
// touches lie in x + [min, max + 1].  reach[s * 8 + d] = max(0, -min over tiles
// of the min offset) and reach[s * 8 + 3 + d] = max(0, max over tiles of the
// max offset + 1): how far below / above itself any voxel of the subject can
// scatter (zeroed before).  Tiles are 32 (d2) x 8 (d1) x 8 (d0).  The squaring
// steps start each box at offsets [-1, 0] and raise a reach from 2 on only: what
// lies within needs no record.
__device__ __forceinline__ void write_record(int mn0, int mn1, int mn2, int mx0, int mx1, int mx2,
                                             int (*red)[ENT / 64], int* __restrict__ boxes,
                                             int s, int tile, int ntiles, int& rmax) {
  mn0 = wave_min(mn0);
  mn1 = wave_min(mn1);
  mn2 = wave_min(mn2);
  mx0 = wave_max(mx0);
  mx1 = wave_max(mx1);
  mx2 = wave_max(mx2);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][w] = mn0;
    red[1][w] = mn1;
    red[2][w] = mn2;
    red[3][w] = mx0;
    red[4][w] = mx1;
    red[5][w] = mx2;
  }
  __syncthreads();
  // thread q < 6 writes entry q of the box and folds its reach into a running
  // maximum (flush_reach issues it once per block): nothing here waits for
  // memory, and no barrier follows, since `red` is rewritten only after the
  // caller's next barrier
  if (threadIdx.x < 6) {
    const int q = threadIdx.x;
    int r = red[q][0];
#pragma unroll
    for (int i = 1; i < ENT / 64; ++i) r = q < 3 ? min(r, red[q][i]) : max(r, red[q][i]);
    boxes[(static_cast<size_t>(s) * ntiles + tile) * 8 + q] = r;
    rmax = max(rmax, q < 3 ? -r : r + 1);
  }
}

// Set and read by blocks of one launch while others do.  A mark that stands is
// not stored again: the stores of a subject's blocks queue up at its line.
__device__ __forceinline__ int get_mark(const int* m) {
  return __hip_atomic_load(m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void set_mark(int* m) {
  if (!get_mark(m)) __hip_atomic_store(m, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The block's reaches into the subject's: thread q < 6 holds entry q.  Atomics
// only where they raise it: those of blocks on one subject queue up at its line
// (k_exp_rec at 16 x 160 x 192 x 160, all subjects flagged: 1.42 ms with every
// tile's, 0.24 with a look first).
__device__ __forceinline__ void flush_reach(int rmax, int* reach, int s) {
  if (threadIdx.x >= 6) return;
  int* r = reach + s * 8 + threadIdx.x;
  if (rmax > get_mark(r)) atomicMax(r, rmax);
}

// Further entries of reach[s * 8 ..], zeroed with the reaches and set by the
// reach-1 adjoint: it met a gradient that is not finite, or too large for it; or
// (CHECK: no records were taken) a cell beyond reach 1, or it did not try.
constexpr int kNonFinite = 6, kFar = 7;

__device__ __forceinline__ int max_reach(const int* rc) {
  return max(max(max(rc[0], rc[1]), max(rc[2], rc[3])), max(rc[4], rc[5]));
}

// Records only, for an adjoint whose forward pass did not take them: of one
// step (flagged: only of the subjects that the reach-1 adjoint left; blocks
// walk the tiles), or of every step (blockIdx.y) of a small launch.  Step t
// reads u_t = src + (t - 1) * fs, step 0 v, scaled.
__global__ __launch_bounds__(ENT) void k_exp_rec(const float* __restrict__ v,
                                                 const float* __restrict__ ckpt, size_t fs, int t0,
                                                 TileGeom tg, float scale, int* __restrict__ boxes,
                                                 size_t box_stride, int* reach,
                                                 size_t reach_stride, bool flagged) {
  __shared__ int red[6][ENT / 64];
  const Geom& g = tg.g;
  const int t = t0 + static_cast<int>(blockIdx.y);
  const float* src = t == 0 ? v : ckpt + static_cast<size_t>(t - 1) * fs;
  const float us = t == 0 ? scale : 1.0f;
  boxes += box_stride * t;
  reach += reach_stride * t;
  const int lx = threadIdx.x % ETX, ly = threadIdx.x / ETX;
  for (uint32_t b = xcd_remap(blockIdx.x, gridDim.x); b < tg.total; b += gridDim.x) {
    const int s = static_cast<int>(b / tg.ntiles);
    const int tile = static_cast<int>(b - static_cast<uint32_t>(s) * tg.ntiles);
    if (flagged && !reach[s * 8 + kNonFinite] && !reach[s * 8 + kFar]) {
      // pass over the rest of this subject's tiles, in whole strides
      const uint32_t rest = static_cast<uint32_t>(s + 1) * tg.ntiles - b;
      b += (rest - 1) / gridDim.x * gridDim.x;
      continue;
    }
    const int ox = tile % tg.ntx * ETX, oy = tile / tg.ntx % tg.nty * ETY,
              oz = tile / (tg.ntx * tg.nty) * ETZ;
    const int x2 = ox + lx, x1 = oy + ly;
    const bool colv = (x2 < g.d2) && (x1 < g.d1);
    const float* f = src + static_cast<size_t>(s) * 3 * g.V;
    int mn0 = INT_MAX, mn1 = INT_MAX, mn2 = INT_MAX, mx0 = INT_MIN, mx1 = INT_MIN, mx2 = INT_MIN;
    for (int k = 0; k < ETZ; ++k) {
      const int x0 = oz + k;
      if (colv && x0 < g.d0) {
        const int lin = (x0 * g.d1 + x1) * g.d2 + x2;
        const BorderCell bc = border_cell(g, x0, x1, x2, f[lin] * us, f[g.V + lin] * us,
                                          f[2 * static_cast<size_t>(g.V) + lin] * us);
        mn0 = min(mn0, bc.i0 - x0);
        mn1 = min(mn1, bc.i1 - x1);
        mn2 = min(mn2, bc.i2 - x2);
        mx0 = max(mx0, bc.i0 - x0);
        mx1 = max(mx1, bc.i1 - x1);
        mx2 = max(mx2, bc.i2 - x2);
      }
    }
    int rmax = 0;
    write_record(mn0, mn1, mn2, mx0, mx1, mx2, red, boxes, s, tile, tg.ntiles, rmax);
    flush_reach(rmax, reach, s);
    __syncthreads();  // `red` is rewritten by the next tile
  }
}

// ---------------------------------------------------------------------------
// Marching kernels: a block owns a column of the (d1, d2) plane, 32 wide, and
// walks a chunk of planes along d0.  A ring of the last planes of u with a halo
// in d1 and d2 lives in LDS; the next plane (of the adjoints also of g) is loaded
// into registers while the current one is computed, so every value is read from
// memory once and loads overlap compute.  Columns of 8 or 16 rows with a
// one-voxel halo for the squaring step (Column below), of 16 for its reach-1
// adjoint, of 8 with a two-voxel halo for the reach-2 adjoint (MarchGeom).
struct MarchGeom {
  TileGeom rec;  // record tiling (the same 32 x 8 columns, 8 planes per record)
  int nzc, tz;   // chunks along d0 and their length (a multiple of ETZ)
  uint32_t total;
};

MarchGeom make_march(const TileGeom& tg, int n, int tz) {
  MarchGeom m;
  m.rec = tg;
  m.tz = tz;
  m.nzc = (tg.g.d0 + tz - 1) / tz;
  m.total = static_cast<uint32_t>(tg.ntx) * tg.nty * m.nzc * n;
  return m;
}

struct MarchId {
  int s, tx, ty, ox, oy, z0, z1;
};

__device__ __forceinline__ MarchId march_id_at(const MarchGeom& m, uint32_t b) {
  MarchId id;
  id.tx = static_cast<int>(b % m.rec.ntx);
  b /= m.rec.ntx;
  id.ty = static_cast<int>(b % m.rec.nty);
  b /= m.rec.nty;
  const int zc = static_cast<int>(b % m.nzc);
  id.s = static_cast<int>(b / m.nzc);
  id.ox = id.tx * ETX;
  id.oy = id.ty * ETY;
  id.z0 = zc * m.tz;
  id.z1 = min(id.z0 + m.tz, m.rec.g.d0);
  return id;
}

// Columns of the marching squaring step and of its reach-1 adjoint: ROWS
// adjacent rows per thread (32 x 8 or 32 x 16 voxels), a one-voxel halo staged
// in LDS.
constexpr int HHX = ETX + 2;
template <int ROWS>
struct Column {
  static constexpr int TY = ROWS * ETY;
  static constexpr int HY = TY + 2;               // staged plane with halo: 34 x 10 or 34 x 18
  static constexpr int HP = HHX * HY;             // 340 or 612 positions
  // One plane of the ring of u, its components HP apart, padded to a multiple
  // of the 64 LDS banks: lanes of a row whose cells lie in different planes then
  // read different banks.
  static constexpr int SLOT = (3 * HP + 63) / 64 * 64;
};
// The adjoint's columns.
constexpr int HTY = Column<2>::TY, HHY = Column<2>::HY, HHP = Column<2>::HP,
              HSLOT = Column<2>::SLOT;
constexpr int HRING = HHP - 2 * ENT;  // its halo positions (100)

struct HatGeom {
  Geom g;
  int ntx, nty, nzc, tz;  // columns and chunks along d0
  uint32_t total;
};

HatGeom make_hat(const TileGeom& tg, int tz, int ty) {
  HatGeom h;
  h.g = tg.g;
  h.ntx = tg.ntx;
  h.nty = (tg.g.d1 + ty - 1) / ty;
  h.tz = tz;
  h.nzc = (tg.g.d0 + tz - 1) / tz;
  h.total = static_cast<uint32_t>(h.ntx) * h.nty * h.nzc * (tg.total / tg.ntiles);
  return h;
}

// Halo-ring position (hy, hx) of thread tid < HRING in the staged plane.
__device__ __forceinline__ void ring_position(int tid, int& hy, int& hx) {
  if (tid < 2 * HHX) {
    hy = tid < HHX ? 0 : HHY - 1;
    hx = tid < HHX ? tid : tid - HHX;
  } else {
    const int q = min(tid - 2 * HHX, 2 * HTY - 1);
    hy = 1 + (q >> 1);
    hx = (q & 1) * (HHX - 1);
  }
}

// As many (discarded) stores after the loads of the loop's first plane as every
// step issues after its loads, so that the wait at the head of the loop counts
// the same on both ways in and leaves the stores in flight.
template <int ROWS>
__device__ __forceinline__ void discarded_stores(const MaskedOut (&out)[3]) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 3 * ROWS; ++k) store_masked(out[k % 3], 0u, 0.0f, false);
  __builtin_amdgcn_sched_barrier(0);
}

// Forward squaring step, marching.  REC: also write the records of the block's
// two record tiles (rows 0-7 and 8-15) per 8 planes.
//
// A stream of 24 B per voxel (read u_t, write u_{t+1}) whose 24 corner reads
// come from LDS; bound by the memory system (1.4x the input fetched, the halo
// lines that L2 no longer holds; neither fewer instructions nor a second plane
// in flight changed its time).  16 x 160 x 192 x 224: 0.60 ms, 4.4 TB/s; on
// 32 x 8 columns with every cell formed in full 0.65.  With |u| < 1 a voxel's cell
// is at -1 or 0 by the sign of u, clamped at the faces by a median; other voxels
// take the general cell, with corners from memory where they leave the staged
// planes.  Records start at offsets [-1, 0] and grow with those other voxels
// only.
template <bool FIRST, bool REC, bool STREAM, int ROWS>
__global__ __launch_bounds__(ENT) void k_exp_fwd(const float* __restrict__ src,
                                                 float* __restrict__ dst, HatGeom m, TileGeom rec,
                                                 float scale, int* __restrict__ boxes,
                                                 int* __restrict__ reach) {
  using C = Column<ROWS>;
  __shared__ float ring[3 * C::SLOT];
  __shared__ int red[6][ENT / 64];
  const Geom& g = m.g;
  uint32_t b = xcd_remap(blockIdx.x, m.total);
  const int tx = static_cast<int>(b % m.ntx);
  b /= m.ntx;
  const int ty = static_cast<int>(b % m.nty);
  b /= m.nty;
  const int z0 = static_cast<int>(b % m.nzc) * m.tz, z1 = min(z0 + m.tz, g.d0);
  const int s = static_cast<int>(b / m.nzc);
  const int ox = tx * ETX, oy = ty * C::TY;
  const size_t off = static_cast<size_t>(s) * 3 * g.V;
  MaskedOut out[3];
  MaskedIn in[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    in[c] = masked_in(src + off + static_cast<size_t>(c) * g.V, static_cast<uint32_t>(g.V));
    out[c] = masked_out(dst + off + static_cast<size_t>(c) * g.V, static_cast<uint32_t>(g.V));
  }
  const int tid = threadIdx.x, lx = tid % ETX, ry = tid / ETX;
  const int x2 = ox + lx, y1 = oy + ROWS * ry;
  const int at = (ROWS * ry + 1) * HHX + lx + 1;  // staged position of the first voxel
  // Staged positions of this thread.  ROWS = 1: tid + j ENT, so that loads run
  // along whole rows with their halo, and rows off the line grid ask once for the
  // lines that they share with it.  ROWS = 2: its own two and, for the first
  // threads, one of the halo ring, so that loads of own rows are whole lines.
  constexpr int NP = (C::HP + ENT - 1) / ENT;
  uint32_t poff[NP];
  int pe[NP];
  const bool last = tid < C::HP - (NP - 1) * ENT;  // the thread has a last position
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    int hy, hx;
    if (ROWS == 1) {
      hy = (tid + j * ENT) / HHX;
      hx = tid + j * ENT - hy * HHX;
    } else if (j < ROWS) {
      hy = 1 + ROWS * ry + j;
      hx = 1 + lx;
    } else {
      ring_position(tid, hy, hx);
    }
    pe[j] = hy * HHX + hx;
    const int y = oy - 1 + hy, x = ox - 1 + hx;
    const bool inside = y >= 0 && y < g.d1 && x >= 0 && x < g.d2 && (j + 1 < NP || last);
    poff[j] = inside ? static_cast<uint32_t>(y * g.d2 + x) << 2 : kNoAccess;
  }
  const float far2 = static_cast<float>(x2 >= g.d2 - 1);  // 1 on the far face, else 0
  const float low2 = x2 > 0 ? -1.0f : 0.0f;
  float pre[NP][3];
  auto load_plane = [&](int z) {  // planes outside the volume are loaded clamped
    const uint32_t zo = static_cast<uint32_t>(min(max(z, 0), g.d0 - 1) * g.plane) << 2;
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int c = 0; c < 3; ++c) pre[j][c] = load_masked(in[c], zo + poff[j]);
  };
  auto stage = [&](int z) {
    float* r = ring + (z + 3) % 3 * C::SLOT;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
      for (int j = 0; j < NP; ++j)
        if (j + 1 < NP || last) r[c * C::HP + pe[j]] = pre[j][c];
    }
  };
  load_plane(z0 - 1);
  stage(z0 - 1);
  load_plane(z0);
  stage(z0);
  load_plane(z0 + 1);
  discarded_stores<ROWS>(out);
  int mn[3] = {-1, -1, -1}, mx[3] = {0, 0, 0};
  int rmax = 0;
  int z = z0;
  do {  // (a loop whose first pass is conditional would let the loads above sink into it)
    stage(z + 1);
    load_plane(z + 2);
    __syncthreads();
    const float* r0 = ring;
    const int slm = (z + 2) % 3 * C::SLOT, slc = z % 3 * C::SLOT, slp = (z + 1) % 3 * C::SLOT;
    const float far0 = static_cast<float>(z >= g.d0 - 1), low0 = z > 0 ? -1.0f : 0.0f;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const int own = at + r * HHX, y = y1 + r;
      const bool live = x2 < g.d2 && y < g.d1;
      float u[3] = {}, res[3] = {};
      if (live) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          u[c] = r0[slc + c * C::HP + own];
          if (FIRST) u[c] *= scale;
        }
        const float far1 = static_cast<float>(y >= g.d1 - 1), low1 = y > 0 ? -1.0f : 0.0f;
        const float w0 = __builtin_amdgcn_fmed3f(u[0], low0, 1.0f - far0),
                    w1 = __builtin_amdgcn_fmed3f(u[1], low1, 1.0f - far1),
                    w2 = __builtin_amdgcn_fmed3f(u[2], low2, 1.0f - far2);
        bool lo0 = w0 < far0, lo1 = w1 < far1, lo2 = w2 < far2;
        float t0 = w0 + (lo0 ? 1.0f : 0.0f), t1 = w1 + (lo1 ? 1.0f : 0.0f),
              t2 = w2 + (lo2 ? 1.0f : 0.0f);
        int pb = own + (lo1 ? -HHX : 0) + (lo2 ? -1 : 0);
        bool ringed = true;
        int base = 0;
        if (!(fabsf(u[0]) < 1.0f && fabsf(u[1]) < 1.0f && fabsf(u[2]) < 1.0f)) {
          const BorderCell bc = border_cell(g, z, y, x2, u[0], u[1], u[2]);
          const int c0 = bc.i0 - z, c1 = bc.i1 - oy + 1, c2 = bc.i2 - ox + 1;
          ringed = c0 >= -1 && c0 <= 0 && c1 >= 0 && c1 + 1 < C::HY && c2 >= 0 && c2 + 1 < HHX;
          lo0 = c0 < 0;
          pb = c1 * HHX + c2;
          base = bc.base;
          t0 = bc.t0;
          t1 = bc.t1;
          t2 = bc.t2;
          if (REC) {
            mn[0] = min(mn[0], c0);
            mn[1] = min(mn[1], bc.i1 - y);
            mn[2] = min(mn[2], bc.i2 - x2);
            mx[0] = max(mx[0], c0);
            mx[1] = max(mx[1], bc.i1 - y);
            mx[2] = max(mx[2], bc.i2 - x2);
          }
        }
        if (ringed) {
          const float* ra = r0 + (pb + (lo0 ? slm : slc));
          const float* rb = r0 + (pb + (lo0 ? slc : slp));
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float cv[8] = {ra[c * C::HP],       ra[c * C::HP + 1],
                                 ra[c * C::HP + HHX], ra[c * C::HP + HHX + 1],
                                 rb[c * C::HP],       rb[c * C::HP + 1],
                                 rb[c * C::HP + HHX], rb[c * C::HP + HHX + 1]};
            res[c] = tri_value(cv, t0, t1, t2);
          }
        } else {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            float cv[8];
            corners_border(src + off + c * static_cast<size_t>(g.V), g, base, cv);
            res[c] = tri_value(cv, t0, t1, t2);
          }
        }
      }
      const uint32_t lin = static_cast<uint32_t>(z * g.plane + y * g.d2 + x2);
#pragma unroll
      for (int c = 0; c < 3; ++c)
        store_masked<STREAM>(out[c], lin, FIRST ? fmaf(res[c], scale, u[c]) : u[c] + res[c], live);
    }
    if (REC && ((z + 1) % ETZ == 0 || z + 1 == z1)) {
      // the box entries over the waves of each record tile (ROWS per column);
      // thread q finishes entry q % 6 of tile q / 6 and folds its reach into a
      // running maximum (issued once per block)
      const int lane = tid & 63, w = tid >> 6;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int a = wave_min(mn[d]), c = wave_max(mx[d]);
        if (lane == 0) {
          red[d][w] = a;
          red[3 + d][w] = c;
        }
        mn[d] = -1;
        mx[d] = 0;
      }
      __syncthreads();
      if (tid < 6 * ROWS) {
        constexpr int NW = ENT / 64 / ROWS;
        const int q = tid % 6, hf = tid / 6;
        int v = red[q][NW * hf];
#pragma unroll
        for (int i = 1; i < NW; ++i)
          v = q < 3 ? min(v, red[q][NW * hf + i]) : max(v, red[q][NW * hf + i]);
        if (oy + ETY * hf < g.d1) {
          const int tile = ((z / ETZ) * rec.nty + ROWS * ty + hf) * rec.ntx + tx;
          boxes[(static_cast<size_t>(s) * rec.ntiles + tile) * 8 + q] = v;
          rmax = max(rmax, q < 3 ? -v : v + 1);
        }
      }
    } else {
      __syncthreads();
    }
  } while (++z < z1);
  if (REC && tid < 6 * ROWS && rmax > 1) atomicMax(reach + s * 8 + tid % 6, rmax);
}

// Adjoint tiles: 4 (d0) x 4 (d1) x 32 (d2) output voxels, two per thread.
constexpr int BTX = 32, BTY = 4, BTZ = 4;
constexpr int BNT = 256;
constexpr int BTILE = BTX * BTY * BTZ;
// cells whose trilinear corners can land in the tile: base index in [O-1, L]
constexpr int CX = BTX + 1, CY = BTY + 1, CZ = BTZ + 1;
constexpr int NCELL = CX * CY * CZ;
constexpr int KSLOT = 2;  // sources kept per cell; further ones take the atomic path

struct BwdGeom {
  TileGeom src;    // tiling of the forward step (its per-tile offsets)
  int ntx, nty, ntz, ntiles;
  uint32_t total;  // adjoint tiles * subjects
};

// Adjoint of one squaring step for one output tile; gout is overwritten.
//
// 1. Each thread keeps the direct term g + J^T g of its two voxels in registers.
// 2. Every source voxel whose cell lies in the tile's cell region takes a slot
//    of that cell (one LDS integer atomic) and stores its fractions and g
//    there; sources beyond KSLOT per cell add their corner contributions to an
//    overflow accumulator with LDS float atomics instead (strong compression
//    only).
// 3. Each thread gathers, for each of its voxels y and each corner offset k,
//    the sources stored in cell y - k with weight w_k.
// LDS of the tiled adjoint.
struct TiledBwdLds {
  int cnt[NCELL];
  float4 sdat4[KSLOT][NCELL];  // t0, t1, t2, g0 of a binned source
  float2 sdat2[KSLOT][NCELL];  // g1, g2
  float ovf[3][BTILE];
  int ubox[6];  // union of the candidate source sub-boxes
};

// One tile of subject s.
template <bool FIRST>
__device__ __forceinline__ void exp_bwd_tile(TiledBwdLds& L, int s, int tile,
                                             const float* __restrict__ ut,
                                             const float* __restrict__ gin,
                                             float* __restrict__ gout, const BwdGeom& bg,
                                             float scale, float oscale,
                                             const int* __restrict__ boxes,
                                             const int* __restrict__ reach) {
  const TileGeom& tg = bg.src;
  const Geom& g = tg.g;
  const int ox = (tile % bg.ntx) * BTX;
  const int oy = ((tile / bg.ntx) % bg.nty) * BTY;
  const int oz = (tile / (bg.ntx * bg.nty)) * BTZ;
  const int L0 = min(oz + BTZ, g.d0) - 1;
  const int L1 = min(oy + BTY, g.d1) - 1;
  const int L2 = min(ox + BTX, g.d2) - 1;
  const int lx = threadIdx.x % BTX, ly = (threadIdx.x / BTX) % BTY, lz = threadIdx.x / (BTX * BTY);
  const size_t off = static_cast<size_t>(s) * 3 * g.V;
  const float* f = ut + off;
  const float* gi = gin + off;
  const float js = FIRST ? scale : 1.0f;

  for (int i = threadIdx.x; i < NCELL; i += BNT) L.cnt[i] = 0;
  for (int i = threadIdx.x; i < 3 * BTILE; i += BNT) (&L.ovf[0][0])[i] = 0.0f;
  if (threadIdx.x < 6) L.ubox[threadIdx.x] = threadIdx.x < 3 ? INT_MAX : INT_MIN;

  // 1. direct term of the two voxels (z = 2 lz, 2 lz + 1) this thread owns
  float acc[2][3];
  const int y1 = oy + ly, y2 = ox + lx;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int y0 = oz + 2 * lz + k;
    acc[k][0] = acc[k][1] = acc[k][2] = 0.0f;
    if (y0 < g.d0 && y1 < g.d1 && y2 < g.d2) {
      const int lin = (y0 * g.d1 + y1) * g.d2 + y2;
      float u0 = f[lin], u1 = f[g.V + lin], u2 = f[2 * g.V + lin];
      if (FIRST) {
        u0 *= scale;
        u1 *= scale;
        u2 *= scale;
      }
      const BorderCell bc = border_cell(g, y0, y1, y2, u0, u1, u2);
      const float gc[3] = {gi[lin], gi[g.V + lin], gi[2 * g.V + lin]};
      float jt0 = 0.0f, jt1 = 0.0f, jt2 = 0.0f;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        float cv[8];
        corners_border(f + c * g.V, g, bc.base, cv);
        const Tri t = tri_eval(cv, bc.t0, bc.t1, bc.t2);
        jt0 += t.d0 * gc[c];
        jt1 += t.d1 * gc[c];
        jt2 += t.d2 * gc[c];
      }
      acc[k][0] = gc[0] + (bc.k0 ? 0.0f : jt0 * js);
      acc[k][1] = gc[1] + (bc.k1 ? 0.0f : jt1 * js);
      acc[k][2] = gc[2] + (bc.k2 ? 0.0f : jt2 * js);
    }
  }
  __syncthreads();

  // 2. bin the source voxels whose cell base lies in [O - 1, L].  A source x
  //    of forward tile s has its cell base in x + [min, max] (the recorded
  //    offsets), so only x_d in [O_d - 1 - max_d, L_d - min_d] can qualify;
  //    candidate forward tiles come from the subject-wide reach (1 where none
  //    is recorded).  The union box of those sub-boxes is swept as one
  //    flattened range, four sources per thread at a time with all their loads
  //    issued before any is used.
  int rc[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) rc[k] = max(reach[s * 8 + k], 1);
  const int lo0 = max(0, oz - rc[3]) / ETZ, hi0 = min(tg.ntz - 1, (L0 + rc[0]) / ETZ);
  const int lo1 = max(0, oy - rc[4]) / ETY, hi1 = min(tg.nty - 1, (L1 + rc[1]) / ETY);
  const int lo2 = max(0, ox - rc[5]) / ETX, hi2 = min(tg.ntx - 1, (L2 + rc[2]) / ETX);
  const int* sbox = boxes + static_cast<size_t>(s) * tg.ntiles * 8;
  {
    const int nc2 = hi2 - lo2 + 1, nc1 = hi1 - lo1 + 1;
    const int ncand = (hi0 - lo0 + 1) * nc1 * nc2;
    for (int ic = threadIdx.x; ic < ncand; ic += BNT) {
      const int sx = lo2 + ic % nc2;
      const int rr = ic / nc2;
      const int sy = lo1 + rr % nc1;
      const int sz = lo0 + rr / nc1;
      const int* bx = sbox + ((sz * tg.nty + sy) * tg.ntx + sx) * 8;
      const int a0 = max(sz * ETZ, oz - 1 - bx[3]);
      const int b0 = min(min(sz * ETZ + ETZ, g.d0) - 1, L0 - bx[0]);
      const int a1 = max(sy * ETY, oy - 1 - bx[4]);
      const int b1 = min(min(sy * ETY + ETY, g.d1) - 1, L1 - bx[1]);
      const int a2 = max(sx * ETX, ox - 1 - bx[5]);
      const int b2 = min(min(sx * ETX + ETX, g.d2) - 1, L2 - bx[2]);
      if (a0 <= b0 && a1 <= b1 && a2 <= b2) {
        atomicMin(&L.ubox[0], a0);
        atomicMin(&L.ubox[1], a1);
        atomicMin(&L.ubox[2], a2);
        atomicMax(&L.ubox[3], b0);
        atomicMax(&L.ubox[4], b1);
        atomicMax(&L.ubox[5], b2);
      }
    }
  }
  __syncthreads();
  const int ua0 = L.ubox[0], ua1 = L.ubox[1], ua2 = L.ubox[2];
  const int ub0 = L.ubox[3], ub1 = L.ubox[4], ub2 = L.ubox[5];
  if (ua0 <= ub0 && ua1 <= ub1 && ua2 <= ub2) {
    const int e2 = ub2 - ua2 + 1, e1 = ub1 - ua1 + 1;
    const int nvox = (ub0 - ua0 + 1) * e1 * e2;
    // q -> (x0, x1, x2) by reciprocal multiplication: for q < 2^23 the FP32
    // product is within one of the exact quotient and is corrected to it;
    // larger boxes use integer division
    const float inv2 = 1.0f / static_cast<float>(e2), inv1 = 1.0f / static_cast<float>(e1);
    const bool small = nvox < (1 << 23);
    for (int qb = 0; qb < nvox; qb += 4 * BNT) {
      float uu[4][3], gg[4][3];
      int xs[4][3];
      bool ok[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = qb + j * BNT + static_cast<int>(threadIdx.x);
        ok[j] = q < nvox;
        const int qq = ok[j] ? q : 0;
        int r, r1;
        if (small) {
          r = static_cast<int>((static_cast<float>(qq) + 0.5f) * inv2);
          r -= (r * e2 > qq);
          r += ((r + 1) * e2 <= qq);
          r1 = static_cast<int>((static_cast<float>(r) + 0.5f) * inv1);
          r1 -= (r1 * e1 > r);
          r1 += ((r1 + 1) * e1 <= r);
        } else {
          r = qq / e2;
          r1 = r / e1;
        }
        xs[j][2] = ua2 + (qq - r * e2);
        xs[j][1] = ua1 + (r - r1 * e1);
        xs[j][0] = ua0 + r1;
        const int lin = (xs[j][0] * g.d1 + xs[j][1]) * g.d2 + xs[j][2];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          uu[j][c] = f[c * g.V + lin];
          gg[j][c] = gi[c * g.V + lin];
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (!ok[j]) continue;
        float u0 = uu[j][0], u1 = uu[j][1], u2 = uu[j][2];
        if (FIRST) {
          u0 *= scale;
          u1 *= scale;
          u2 *= scale;
        }
        const BorderCell bc = border_cell(g, xs[j][0], xs[j][1], xs[j][2], u0, u1, u2);
        // local cell index: base - (O - 1), in [0, C)
        const int c0 = bc.i0 - oz + 1, c1 = bc.i1 - oy + 1, c2 = bc.i2 - ox + 1;
        if (c0 < 0 || c0 >= CZ || c1 < 0 || c1 >= CY || c2 < 0 || c2 >= CX) continue;
        const int ci = (c0 * CY + c1) * CX + c2;
        const float g0 = gg[j][0], g1 = gg[j][1], g2 = gg[j][2];
        const int slot = atomicAdd(&L.cnt[ci], 1);
        if (slot < KSLOT) {
          L.sdat4[slot][ci] = make_float4(bc.t0, bc.t1, bc.t2, g0);
          L.sdat2[slot][ci] = make_float2(g1, g2);
        } else {
          const float w0[2] = {1.0f - bc.t0, bc.t0};
          const float w1[2] = {1.0f - bc.t1, bc.t1};
          const float w2[2] = {1.0f - bc.t2, bc.t2};
#pragma unroll
          for (int a = 0; a < 2; ++a) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                // corner (c + k) - 1 in tile-local coordinates
                const int q0 = c0 + a - 1, q1 = c1 + b - 1, q2 = c2 + e - 1;
                if (q0 >= 0 && q0 < BTZ && q1 >= 0 && q1 < BTY && q2 >= 0 && q2 < BTX) {
                  const float w = w0[a] * w1[b] * w2[e];
                  const int li = (q0 * BTY + q1) * BTX + q2;
                  atomicAdd(&L.ovf[0][li], w * g0);
                  atomicAdd(&L.ovf[1][li], w * g1);
                  atomicAdd(&L.ovf[2][li], w * g2);
                }
              }
            }
          }
        }
      }
    }
  }
  __syncthreads();

  // 3. gather: voxel y receives w_k(x) g(x) from every source x binned in
  //    cell y - k, k in {0,1}^3
  float* go = gout + off;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int z = 2 * lz + k;
    const int y0 = oz + z;
    if (!(y0 < g.d0 && y1 < g.d1 && y2 < g.d2)) continue;
    float r0 = acc[k][0], r1 = acc[k][1], r2 = acc[k][2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int ci = ((z + 1 - a) * CY + (ly + 1 - b)) * CX + (lx + 1 - e);
          const int nsrc = min(L.cnt[ci], KSLOT);
#pragma unroll
          for (int j = 0; j < KSLOT; ++j) {
            if (j < nsrc) {
              const float4 p = L.sdat4[j][ci];
              const float2 q = L.sdat2[j][ci];
              const float w = corner_weight(a, b, e, p.x, p.y, p.z);
              r0 += w * p.w;
              r1 += w * q.x;
              r2 += w * q.y;
            }
          }
        }
      }
    }
    const int li = (z * BTY + ly) * BTX + lx;
    r0 += L.ovf[0][li];
    r1 += L.ovf[1][li];
    r2 += L.ovf[2][li];
    const int lin = (y0 * g.d1 + y1) * g.d2 + y2;
    go[lin] = r0 * oscale;
    go[g.V + lin] = r1 * oscale;
    go[2 * g.V + lin] = r2 * oscale;
  }
  __syncthreads();  // the next tile reuses the LDS bins
}

// Adjoint of one squaring step, marching, for a subject whose every cell
// offset lies in [-1, 0] (reach 1 in every direction: all |u_t| < 1, the
// case of the early sweeps and of the first squaring steps).
//
// With |u| <= 1 the trilinear weight of source x on target y is a product of
// hat functions, prod_d max(0, 1 - |x_d + u_d - y_d|), and along each axis the
// hat at target offset +1, 0, -1 is max(u, 0), 1 - |u|, max(-u, 0): one
// instruction from the source's displacement, no cell, no bin.  A target
// gathers from the 3 x 3 x 3 sources around it.  Marching over source planes
// q, each target column sums over the 9 in-plane sources, w their in-plane
// weight,
//   S0 = sum w g,  Sa = sum w |u0| g,  Ss = sum w u0 g,
// which give the plane's contributions to target planes q (S0 - Sa), q + 1
// ((Sa + Ss) / 2) and q - 1 ((Sa - Ss) / 2); a target is complete once its
// plane, the one before and the one after have been walked, and its partial
// sums stay in registers.
//
// Bound by vector issue: about 290 vector instructions per voxel at 85 % of
// the issue slots, 6 TB/s out of L2 beside it.  The 9 pairs take 12
// instructions each; threads own two adjacent rows of a 32 x 16 column, so
// that a source read from LDS serves up to six pairs and the staged halo is
// 1.2x the tile.  16 x 160 x 192 x 224, one step: 1.17 ms; binning the sources
// by cell instead (an LDS atomic and 24 bytes written per source, two slots of
// four cells read per target, the bins cleared per plane, 32 x 8 columns: 362
// vector instructions) took 1.40 ms.  16 x 160 x 192 x 160: 0.76 and 0.95 ms.
//
// Border clamping moves a source whose position leaves the volume onto its
// face: the staged u of the two layers at a face is clamped to what stays inside
// (a voxel there may point outwards by any amount and still have its cell within
// reach 1).  Positions outside the volume are staged with
// g = 0.
//
// A source contributes to the eight corners of its cell only, so a target
// next to it must not see 0 * g when g is not finite; and the doubled sums of up
// to 27 sources must not leave the range of FP32 where the gradient does not.  A
// block that meets a g that is not finite or beyond kHatMax says so in its
// subject's record (kNonFinite), and the reach-2 kernel, launched after this
// one, then computes that subject again.
constexpr float kHatMax = 0x1p120f;
struct HatLds {
  float uring[3 * HSLOT];  // u_t of planes q-2, q-1, q (slot p % 3)
  float4 src4[HHP];        // plane q: clamped u (scaled in the first step), g0
  float2 src2[HHP];        // g1, g2
  int skip;                // the block has nothing to do
  int stop;                // a cell beyond reach 1 was staged
};

// Hat function of a displacement u at target offset d (-1, 0 or 1), |u| <= 1.
__device__ __forceinline__ float hat(float u, int d) {
  return d == 0 ? 1.0f - fabsf(u) : __builtin_amdgcn_fmed3f(d > 0 ? u : -u, 0.0f, 1.0f);
}

// Sums over the in-plane sources of plane q for the two targets whose first
// source is staged at `at` (two rows of one column).
__device__ __forceinline__ void hat_pairs(const HatLds& L, int at, float (&s0)[2][3],
                                          float (&sa)[2][3], float (&ss)[2][3]) {
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) s0[r][c] = sa[r][c] = ss[r][c] = 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const float4 p = L.src4[at + j * HHX + i];
      const float2 q = L.src2[at + j * HHX + i];
      // the source lies i - 1 columns and j - 1 - r rows from the target
      const float hx = hat(p.z, 1 - i);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int dy = r + 1 - j;
        if (dy < -1 || dy > 1) continue;
        const float w = hx * hat(p.y, dy), wz = w * p.x;
        s0[r][0] = fmaf(w, p.w, s0[r][0]);
        s0[r][1] = fmaf(w, q.x, s0[r][1]);
        s0[r][2] = fmaf(w, q.y, s0[r][2]);
        sa[r][0] = fmaf(fabsf(wz), p.w, sa[r][0]);
        sa[r][1] = fmaf(fabsf(wz), q.x, sa[r][1]);
        sa[r][2] = fmaf(fabsf(wz), q.y, sa[r][2]);
        ss[r][0] = fmaf(wz, p.w, ss[r][0]);
        ss[r][1] = fmaf(wz, q.x, ss[r][1]);
        ss[r][2] = fmaf(wz, q.y, ss[r][2]);
      }
    }
  }
}

// Range of the displacement along one axis that stays inside the volume, as
// two bytes (-lo, hi), each at most 2: a position within reach 1 is clamped to
// [x + lo, x + hi].
__device__ __forceinline__ uint32_t hat_range(int x, int D) {
  return static_cast<uint32_t>(min(max(x, 0), 2)) |
         (static_cast<uint32_t>(min(max(D - 1 - x, 0), 2)) << 8);
}
__device__ __forceinline__ float hat_clamp(float u, uint32_t range) {
  return __builtin_amdgcn_fmed3f(u, -static_cast<float>(range & 255u),
                                 static_cast<float>((range >> 8) & 255u));
}
// Whether the cell of a displacement, clamped near the faces, lies beyond reach
// 1.  (One voxel before the far face a clamped +1 lies in the last cell, at
// fraction 1; a NaN points to the low face, as everywhere.)
__device__ __forceinline__ bool hat_beyond(float w, uint32_t range) {
  return !(w >= -1.0f) || (w >= 1.0f && ((range >> 8) & 255u) == 2u);
}

// CHECK: the forward took no records.  The kernel then looks at the
// displacements it stages; a block that meets a cell beyond reach 1 marks the
// subject (kFar) and ends, and the records of marked subjects are taken
// afterwards for the other adjoints.  `later` (or NULL) are the reaches of the
// step after this one, walked before it: a subject with a reach of 4 or more
// there is marked without a try, since a step of reach 1 gives one of at most 2
// (two displacements in [-1, 1) add up to one in [-2, 2); more than one voxel
// outwards occurs only beside a face, where the clamped cells stay within 2).
template <bool FIRST, bool CHECK, bool STREAM>
__global__ __launch_bounds__(ENT, 4) void k_exp_bwd_hat(const float* __restrict__ ut,
                                                        const float* __restrict__ gin,
                                                        float* __restrict__ gout, HatGeom m,
                                                        float scale, float oscale,
                                                        int* __restrict__ reach,
                                                        const int* __restrict__ later) {
  __shared__ HatLds L;
  const Geom& g = m.g;
  uint32_t b = xcd_remap(blockIdx.x, m.total);
  const int ox = static_cast<int>(b % m.ntx) * ETX;
  b /= m.ntx;
  const int oy = static_cast<int>(b % m.nty) * HTY;
  b /= m.nty;
  const int z0 = static_cast<int>(b % m.nzc) * m.tz, z1 = min(z0 + m.tz, g.d0);
  const int s = static_cast<int>(b / m.nzc);
  if (CHECK) {
    // one thread reads the mark, which other blocks set meanwhile, for all
    if (threadIdx.x == 0) {
      const bool tried = !later || max_reach(later + s * 8) < 4;
      if (!tried && ox == 0 && oy == 0 && z0 == 0) set_mark(reach + s * 8 + kFar);
      L.skip = !tried || get_mark(reach + s * 8 + kFar);
      L.stop = 0;
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(L.skip)) return;
  } else if (max_reach(reach + s * 8) > 1) {
    return;
  }
  const size_t off = static_cast<size_t>(s) * 3 * g.V;
  MaskedOut out[3];
#pragma unroll
  for (int c = 0; c < 3; ++c)
    out[c] = masked_out(gout + off + static_cast<size_t>(c) * g.V, static_cast<uint32_t>(g.V));
  const int tid = threadIdx.x, lx = tid % ETX, ry = tid / ETX;
  const float js = FIRST ? 2.0f * scale : 2.0f;  // sums are kept doubled (see the update below)
  const float os = 0.5f * oscale;

  // Staged positions of this thread: its two targets (rows 2 ry and 2 ry + 1)
  // and, for the first HRING threads, one of the halo ring.  Positions outside
  // the volume (and threads without a ring position) load past the range
  // check and get zeros.
  const int at0 = 2 * ry * HHX + lx;  // staged position of the first target's first source
  const int x2 = ox + lx, y1 = oy + 2 * ry;
  int pr;                 // the ring position
  uint32_t poff[3];       // byte offsets within a plane
  uint32_t prange[3];     // clamping ranges along d2 and d1
  {
    int hy, hx;
    ring_position(tid, hy, hx);
    pr = hy * HHX + hx;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int y = j < 2 ? y1 + j : oy - 1 + hy, x = j < 2 ? x2 : ox - 1 + hx;
      const bool in = y >= 0 && y < g.d1 && x >= 0 && x < g.d2 && (j < 2 || tid < HRING);
      poff[j] = in ? static_cast<uint32_t>(y * g.d2 + x) << 2 : kNoAccess;
      prange[j] = hat_range(x, g.d2) | (hat_range(y, g.d1) << 16);
    }
  }
  const bool ring = tid < HRING;
  // the tile or its halo touches the two outer layers of the volume in d1 or d2
  const bool face = oy == 0 || ox == 0 || oy + HTY >= g.d1 - 2 || ox + ETX >= g.d2 - 2;

  float pu[3][3], pg[3][3];
  auto load_plane = [&](int z) {
    // a plane outside the volume: nothing is in range
    const uint32_t zo = static_cast<uint32_t>(min(max(z, 0), g.d0 - 1) * g.plane) << 2;
    const uint32_t count = z >= 0 && z < g.d0 ? static_cast<uint32_t>(g.V) : 0u;
    MaskedIn fu[3], fg[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const size_t oc = off + static_cast<size_t>(c) * g.V;
      fu[c] = masked_in(ut + oc, count);
      fg[c] = masked_in(gin + oc, count);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        pu[j][c] = load_masked(fu[c], zo + poff[j]);
        pg[j][c] = load_masked(fg[c], zo + poff[j]);
      }
  };
  bool bad = false;  // a g that is not finite, or too large, was staged
  auto stage = [&](int z) {
    const int sl = (z + 3) % 3;
    const uint32_t rz = hat_range(z, g.d0);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      if (j == 2 && !ring) continue;
      // LDS offsets recomputed on every plane: held in registers they would
      // cost the fourth wave per SIMD
      int e = j < 2 ? at0 + (j + 1) * HHX + 1 : pr;
      asm volatile("" : "+v"(e));
      float u[3] = {pu[j][0], pu[j][1], pu[j][2]};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        L.uring[sl * HSLOT + c * HHP + e] = u[c];
        if (FIRST) u[c] *= scale;
      }
      if (face || z <= 1 || z >= g.d0 - 2) {
        u[0] = hat_clamp(u[0], rz);
        u[1] = hat_clamp(u[1], prange[j] >> 16);
        u[2] = hat_clamp(u[2], prange[j]);
      }
      // (the ring's voxels are other columns' own)
      if (CHECK && j < 2 && !(fabsf(u[0]) < 1.0f && fabsf(u[1]) < 1.0f && fabsf(u[2]) < 1.0f)) {
        if (hat_beyond(u[0], rz) || hat_beyond(u[1], prange[j] >> 16) ||
            hat_beyond(u[2], prange[j]))
          L.stop = 1;
      }
      bad |= !(fabsf(pg[j][0]) + fabsf(pg[j][1]) + fabsf(pg[j][2]) < kHatMax);
      L.src4[e] = make_float4(u[0], u[1], u[2], pg[j][0]);
      L.src2[e] = make_float2(pg[j][1], pg[j][2]);
    }
  };

  load_plane(z0 - 1);
  discarded_stores<2>(out);
  // twice the partial sums of the targets of planes q - 1 and q
  float accA[2][3] = {}, accB[2][3] = {};
  float og[2][3] = {};  // g of the targets of plane q - 1
  int q = z0 - 1;
  do {
    stage(q);
    load_plane(q + 1);
    __syncthreads();
    if (CHECK && __builtin_amdgcn_readfirstlane(L.stop)) {
      if (tid == 0) set_mark(reach + s * 8 + kFar);
      return;
    }
    const int p = q - 1;  // the target plane finished by this step
    int at = at0;
    asm volatile("" : "+v"(at));
    if (p >= z0) {
      // ring slots (as offsets) of planes p-1, p, p+1
      const int slm = (p + 2) % 3 * HSLOT, slc = p % 3 * HSLOT, slp = (p + 1) % 3 * HSLOT;
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        // direct term: J^T g = gradient of the interpolant of g . u at the
        // sample, corners from the ring
        const int own = at + (r + 1) * HHX + 1;
        float u[3];
        bool lo[3], kl[3] = {false, false, false};  // cell below x; clamped
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          u[c] = L.uring[slc + c * HHP + own];
          if (FIRST) u[c] *= scale;
          lo[c] = u[c] < 0.0f;
        }
        if (face || p <= 1 || p >= g.d0 - 2) {
          // clamped positions, the last cell at the far faces, no derivative
          // along a clamped axis
          const uint32_t rg[3] = {hat_range(p, g.d0), prange[r] >> 16, prange[r]};
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float w = hat_clamp(u[c], rg[c]);
            kl[c] = w != u[c];
            u[c] = w;
            lo[c] = w < (((rg[c] >> 8) & 255u) ? 0.0f : 1.0f);
          }
        }
        const float f0 = u[0] + (lo[0] ? 1.0f : 0.0f), f1 = u[1] + (lo[1] ? 1.0f : 0.0f),
                    f2 = u[2] + (lo[2] ? 1.0f : 0.0f);
        // one component's corners: rows of planes i0 and i0 + 1
        const int pb = own + (lo[1] ? -HHX : 0) + (lo[2] ? -1 : 0);
        const float* ra = L.uring + (pb + (lo[0] ? slm : slc));
        const float* rb = L.uring + (pb + (lo[0] ? slc : slp));
        float h[8];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float cv[8] = {ra[c * HHP],       ra[c * HHP + 1],
                               ra[c * HHP + HHX], ra[c * HHP + HHX + 1],
                               rb[c * HHP],       rb[c * HHP + 1],
                               rb[c * HHP + HHX], rb[c * HHP + HHX + 1]};
#pragma unroll
          for (int k = 0; k < 8; ++k) h[k] = c == 0 ? og[r][0] * cv[k] : h[k] + og[r][c] * cv[k];
        }
        const Tri t = tri_eval(h, f0, f1, f2);
        const float d[3] = {kl[0] ? 0.0f : t.d0, kl[1] ? 0.0f : t.d1, kl[2] ? 0.0f : t.d2};
#pragma unroll
        for (int c = 0; c < 3; ++c)
          accA[r][c] = fmaf(js, d[c], fmaf(2.0f, og[r][c], accA[r][c]));
      }
    }
    float s0[2][3], sa[2][3], ss[2][3];
    hat_pairs(L, at, s0, sa, ss);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int own = at + (r + 1) * HHX + 1;
      const float2 b2 = L.src2[own];
      og[r][0] = L.src4[own].w;
      og[r][1] = b2.x;
      og[r][2] = b2.y;
    }
    // plane q's parts, doubled: sa - ss of targets q - 1 (now complete),
    // 2 (s0 - sa) of targets q, sa + ss of targets q + 1.  Range-checked
    // stores on every plane: a store under a branch would make the next
    // staging wait for it together with the plane in flight.
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const uint32_t lin = static_cast<uint32_t>(p * g.plane + (y1 + r) * g.d2 + x2);
      const bool on = p >= z0 && x2 < g.d2 && y1 + r < g.d1;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        store_masked<STREAM>(out[c], lin, (accA[r][c] + (sa[r][c] - ss[r][c])) * os, on);
        accA[r][c] = fmaf(2.0f, s0[r][c] - sa[r][c], accB[r][c]);
        accB[r][c] = sa[r][c] + ss[r][c];
      }
    }
    __syncthreads();
  } while (++q <= z1);
  if (bad) set_mark(reach + s * 8 + kNonFinite);
}

// The same gather without marching, for volumes too small to fill the chip with
// columns: a block owns 32 x 8 x 2 targets (two per thread, along d0), stages
// the 34 x 10 x 4 sources around them at once and every thread sums over its
// 3 x 3 x 4.  Bound by latency (one load round, one barrier, about 550 vector
// instructions per wave at a wave or two per SIMD): tiles of 512 targets give
// 4 x 32^3 one block per CU.  A subject with a larger reach takes the binning
// tile in the same launch (an idle launch would cost a third of this kernel).
// 4 x 32^3, one step: 6.4 us; the binning tile for every subject took 12.7 us.
constexpr int NTY = 8, NTZ = 2;                       // rows and planes of a tile
constexpr int NHY = NTY + 2, NHZ = NTZ + 2;
constexpr int NHP = HHX * NHY * NHZ;                  // 1360 staged positions
constexpr int NNJ = (NHP + ENT - 1) / ENT;            // per thread (6)

struct NearLds {
  float uraw[3][NHP];  // u_t
  float4 src4[NHP];    // clamped u (scaled in the first step), g0
  float2 src2[NHP];    // g1, g2
  int nonfinite;
};

struct NearGeom {
  BwdGeom bg;                // the binning tiles
  int nty, ntz;              // near tiles (as many along d2 as bg)
  int items;                 // blocks per subject: the larger of the two counts
};

NearGeom make_near(const BwdGeom& bg) {
  NearGeom ng;
  ng.bg = bg;
  ng.nty = (bg.src.g.d1 + NTY - 1) / NTY;
  ng.ntz = (bg.src.g.d0 + NTZ - 1) / NTZ;
  const int near = bg.ntx * ng.nty * ng.ntz;
  ng.items = near > bg.ntiles ? near : bg.ntiles;
  return ng;
}

template <bool FIRST>
__device__ __forceinline__ void exp_bwd_near(NearLds& L, int s, int tile,
                                             const float* __restrict__ ut,
                                             const float* __restrict__ gin,
                                             float* __restrict__ gout, const NearGeom& ng,
                                             float scale, float oscale) {
  const Geom& g = ng.bg.src.g;
  const int ox = (tile % ng.bg.ntx) * ETX;
  const int oy = (tile / ng.bg.ntx) % ng.nty * NTY;
  const int oz = tile / (ng.bg.ntx * ng.nty) * NTZ;
  const size_t off = static_cast<size_t>(s) * 3 * g.V;
  const int tid = threadIdx.x;
  if (tid == 0) L.nonfinite = 0;
  __syncthreads();
  float pu[NNJ][3], pg[NNJ][3];
#pragma unroll
  for (int j = 0; j < NNJ; ++j) {
    const int e = tid + j * ENT;
    const int hz = e / (HHX * NHY), r = e - hz * (HHX * NHY);
    const int hy = r / HHX, hx = r - hy * HHX;
    const int z = oz - 1 + hz, y = oy - 1 + hy, x = ox - 1 + hx;
    const bool in = e < NHP && z >= 0 && z < g.d0 && y >= 0 && y < g.d1 && x >= 0 && x < g.d2;
    const uint32_t lin = in ? static_cast<uint32_t>((z * g.d1 + y) * g.d2 + x) << 2 : kNoAccess;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const size_t oc = off + static_cast<size_t>(c) * g.V;
      pu[j][c] = load_masked(masked_in(ut + oc, static_cast<uint32_t>(g.V)), lin);
      pg[j][c] = load_masked(masked_in(gin + oc, static_cast<uint32_t>(g.V)), lin);
    }
  }
#pragma unroll
  for (int j = 0; j < NNJ; ++j) {
    const int e = tid + j * ENT;
    if (e >= NHP) continue;
    const int hz = e / (HHX * NHY), r = e - hz * (HHX * NHY);
    const int hy = r / HHX, hx = r - hy * HHX;
    const float js = FIRST ? scale : 1.0f;
    L.src4[e] = make_float4(hat_clamp(pu[j][0] * js, hat_range(oz - 1 + hz, g.d0)),
                            hat_clamp(pu[j][1] * js, hat_range(oy - 1 + hy, g.d1)),
                            hat_clamp(pu[j][2] * js, hat_range(ox - 1 + hx, g.d2)), pg[j][0]);
    L.src2[e] = make_float2(pg[j][1], pg[j][2]);
#pragma unroll
    for (int c = 0; c < 3; ++c) L.uraw[c][e] = pu[j][c];
    if (!__builtin_isfinite(pg[j][0] + pg[j][1] + pg[j][2])) L.nonfinite = 1;
  }
  __syncthreads();
  const int lx = tid % ETX, ly = tid / ETX;
  const int at = ly * HHX + lx;  // first of the sources around the first target
  float acc[2][3] = {};
  if (!L.nonfinite) {
#pragma unroll
    for (int k = 0; k < NHZ; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const float4 p = L.src4[at + (k * NHY + j) * HHX + i];
          const float2 q = L.src2[at + (k * NHY + j) * HHX + i];
          const float w = hat(p.y, 1 - j) * hat(p.z, 1 - i);
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            if (r + 1 - k < -1 || r + 1 - k > 1) continue;
            const float wt = w * hat(p.x, r + 1 - k);
            acc[r][0] = fmaf(wt, p.w, acc[r][0]);
            acc[r][1] = fmaf(wt, q.x, acc[r][1]);
            acc[r][2] = fmaf(wt, q.y, acc[r][2]);
          }
        }
  } else {
    // a gradient that is not finite reaches the eight corners of its cell
    // (whatever their weight) and nothing else
#pragma unroll 1
    for (int e = 0; e < 9 * NHZ; ++e) {
      const int k = e / 9, j = e / 3 % 3, i = e % 3;
      const float4 p = L.src4[at + (k * NHY + j) * HHX + i];
      const float2 q = L.src2[at + (k * NHY + j) * HHX + i];
      const int o0 = (p.x < 0.0f || oz + k - 1 == g.d0 - 1) ? -1 : 0;
      const int o1 = (p.y < 0.0f || oy + ly + j - 1 == g.d1 - 1) ? -1 : 0;
      const int o2 = (p.z < 0.0f || ox + lx + i - 1 == g.d2 - 1) ? -1 : 0;
      const int e1 = 1 - j - o1, e2 = 1 - i - o2;
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int e0 = r + 1 - k - o0;
        if (((e0 | e1 | e2) & ~1) != 0) continue;
        const float wt = corner_weight(e0, e1, e2, p.x - o0, p.y - o1, p.z - o2);
        acc[r][0] += wt * p.w;
        acc[r][1] += wt * q.x;
        acc[r][2] += wt * q.y;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int z = oz + r, y = oy + ly, x = ox + lx;
    // direct term (computed for ragged lanes too, from staged zeros)
    const int own = at + ((r + 1) * NHY + 1) * HHX + 1;
    const float4 p = L.src4[own];
    const float2 q = L.src2[own];
    const float js = FIRST ? scale : 1.0f;
    const bool k0 = L.uraw[0][own] * js != p.x, k1 = L.uraw[1][own] * js != p.y,
               k2 = L.uraw[2][own] * js != p.z;
    const int o0 = (p.x < 0.0f || z == g.d0 - 1) ? 1 : 0;
    const int o1 = (p.y < 0.0f || y == g.d1 - 1) ? 1 : 0;
    const int o2 = (p.z < 0.0f || x == g.d2 - 1) ? 1 : 0;
    const int pb = own - (o0 * NHY + o1) * HHX - o2;
    const float gc[3] = {p.w, q.x, q.y};
    float h[8];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float cv = L.uraw[c][pb + ((k >> 2) * NHY + ((k >> 1) & 1)) * HHX + (k & 1)];
        h[k] = c == 0 ? gc[0] * cv : h[k] + gc[c] * cv;
      }
    const Tri t = tri_eval(h, p.x + o0, p.y + o1, p.z + o2);
    if (z < g.d0 && y < g.d1 && x < g.d2) {
      float* o = gout + off;
      const uint32_t lin = static_cast<uint32_t>((z * g.d1 + y) * g.d2 + x);
      st_at(o, lin, (acc[r][0] + gc[0] + (k0 ? 0.0f : t.d0 * js)) * oscale);
      st_at(o + g.V, lin, (acc[r][1] + gc[1] + (k1 ? 0.0f : t.d1 * js)) * oscale);
      st_at(o + 2 * static_cast<size_t>(g.V), lin,
            (acc[r][2] + gc[2] + (k2 ? 0.0f : t.d2 * js)) * oscale);
    }
  }
}

union SmallBwdLds {
  TiledBwdLds tiled;
  NearLds near;
};

template <bool FIRST>
__global__ __launch_bounds__(ENT) void k_exp_bwd_small(const float* __restrict__ ut,
                                                       const float* __restrict__ gin,
                                                       float* __restrict__ gout, NearGeom ng,
                                                       float scale, float oscale,
                                                       const int* __restrict__ boxes,
                                                       const int* __restrict__ reach) {
  __shared__ __align__(16) unsigned char lds[sizeof(SmallBwdLds)];
  SmallBwdLds& L = *reinterpret_cast<SmallBwdLds*>(lds);
  const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
  const int s = static_cast<int>(b / ng.items);
  const int item = static_cast<int>(b - static_cast<uint32_t>(s) * ng.items);
  const int* rc = reach + s * 8;
  if (max(max(max(rc[0], rc[1]), max(rc[2], rc[3])), max(rc[4], rc[5])) <= 1) {
    if (item < ng.bg.ntx * ng.nty * ng.ntz)
      exp_bwd_near<FIRST>(L.near, s, item, ut, gin, gout, ng, scale, oscale);
  } else if (item < ng.bg.ntiles) {
    exp_bwd_tile<FIRST>(L.tiled, s, item, ut, gin, gout, ng.bg, scale, oscale, boxes, reach);
  }
}

// Adjoint of one squaring step, marching, for a subject whose cell offsets
// lie in [-2, 1] on every axis (reach 2: roughly 1 <= max |u_t| < 2, the later
// squaring steps of moderate deformations; and the subjects within [-1, 0] that
// the reach-1 kernel leaves).  Sources are binned by cell, one cell plane live at a time: a
// source of plane p falls in cell planes p-2 .. p+1, so cell plane z is filled from
// the sources of planes z-1 .. z+2, whose cells are computed once, when their
// plane is staged, and kept in registers for four iterations; sources up to
// two voxels outside the column can land in its cell region (a two-voxel halo
// ring of 176 positions, one for each of the first 176 threads); the direct
// term's corners lie in planes z-2 .. z+2 of the u ring.  Iteration z:
// (i) clear the cell plane and target plane z+1's overflow, stage u of plane
// z+2 and compute its sources' cells; (ii) bin the sources of planes
// z-1 .. z+2 whose cell lies in plane z; (iii) the direct term of the plane-z
// targets; (iv) the gather, finishing plane z and starting plane z+1.
constexpr int MCX = ETX + 1, MCY = ETY + 1;  // cells per cell plane: 33 x 9
constexpr int MCP = MCX * MCY;
constexpr int H2X = ETX + 4, H2Y = ETY + 4;  // staged plane with a two-voxel halo: 36 x 12
constexpr int H2P = H2X * H2Y;               // 432 positions
constexpr int H2RING = H2P - ENT;            // 176 halo positions

// One source: its cell packed as r2 (6 bits: corner column in the staged
// plane), r1 (4 bits: corner row), o0 + 2 (2 bits: cell plane - source
// plane + 2), the three clamped flags and a valid bit (the source exists and
// its cell's corners lie in the staged plane); fractions and g.
struct Src2 {
  int key;
  float t0, t1, t2, g0, g1, g2;
};
constexpr int kSrcValid = 1 << 15;

struct March2Lds {
  float uring[5][3][H2P];  // u_t of planes z-2 .. z+2 (slot p % 5)
  int bcnt[MCP];           // the live cell plane
  float4 bd4[KSLOT][MCP];  // t0, t1, t2, g0 per binned source (0 if empty)
  float2 bd2[KSLOT][MCP];  // g1, g2
  float ovf[2][3][ENT];    // overflow into target planes, by parity
};

// One chunk of one column.
template <bool FIRST>
__device__ __forceinline__ void exp_bwd_march2(March2Lds& L, const MarchGeom& m, const MarchId& id,
                                               const float* __restrict__ ut,
                                               const float* __restrict__ gin,
                                               float* __restrict__ gout, float scale,
                                               float oscale) {
  auto& uring = L.uring;
  auto& bcnt = L.bcnt;
  auto& bd4 = L.bd4;
  auto& bd2 = L.bd2;
  auto& ovf = L.ovf;
  const Geom& g = m.rec.g;
  const size_t off = static_cast<size_t>(id.s) * 3 * g.V;
  const float* f = ut + off;
  const float* gi = gin + off;
  float* go = gout + off;
  const int lx = threadIdx.x % ETX, ly = threadIdx.x / ETX;
  const float js = FIRST ? scale : 1.0f;

  // staged positions: j = 0 the thread's own voxel, j = 1 a halo-ring voxel
  int pe[2], py[2], px[2], poff[2];
  bool puse[2], pin[2];
  pe[0] = (ly + 2) * H2X + lx + 2;
  py[0] = id.oy + ly;
  px[0] = id.ox + lx;
  puse[0] = true;
  {
    const int r = threadIdx.x;
    int hy, hx;
    if (r < 2 * H2X) {  // rows 0 and 1
      hy = r / H2X;
      hx = r - hy * H2X;
    } else if (r < 4 * H2X) {  // rows H2Y - 2 and H2Y - 1
      const int q = r - 2 * H2X;
      hy = H2Y - 2 + q / H2X;
      hx = q - (q / H2X) * H2X;
    } else {  // columns 0, 1, H2X - 2, H2X - 1 of rows 2 .. H2Y - 3
      const int q = min(r - 4 * H2X, 4 * ETY - 1);
      hy = 2 + q / 4;
      const int col = q % 4;
      hx = col < 2 ? col : H2X - 4 + col;
    }
    puse[1] = r < H2RING;
    pe[1] = hy * H2X + hx;
    py[1] = id.oy - 2 + hy;
    px[1] = id.ox - 2 + hx;
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    pin[j] = py[j] >= 0 && py[j] < g.d1 && px[j] >= 0 && px[j] < g.d2;
    poff[j] = min(max(py[j], 0), g.d1 - 1) * g.d2 + min(max(px[j], 0), g.d2 - 1);
  }
  if (!puse[1]) poff[1] = poff[0];

  const float* fc[3] = {f, f + g.V, f + 2 * static_cast<size_t>(g.V)};
  const float* gc[3] = {gi, gi + g.V, gi + 2 * static_cast<size_t>(g.V)};
  // the next plane to stage in flight (every lane loads, planes past the
  // volume clamped; a second buffer measured slower at this register count)
  float pu[2][3], pg[2][3];
  auto load_plane = [&](int z, float (&lu)[2][3], float (&lg)[2][3]) {
    const int zc = min(max(z, 0), g.d0 - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t lin = static_cast<uint32_t>(zc * g.plane + poff[j]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lu[j][c] = ld_at(fc[c], lin);
        lg[j][c] = ld_at(gc[c], lin);
      }
    }
  };
  auto store_u = [&](int z, const float (&su_)[2][3]) {
    const int sl = (z + 10) % 5;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (puse[j]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) uring[sl][c][pe[j]] = su_[j][c];
      }
  };
  auto clear_cells = [&]() {
    const float4 z4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const float2 z2 = make_float2(0.0f, 0.0f);
    for (int i = threadIdx.x; i < MCP; i += ENT) {
      bcnt[i] = 0;
#pragma unroll
      for (int k = 0; k < KSLOT; ++k) {
        bd4[k][i] = z4;
        bd2[k][i] = z2;
      }
    }
  };
  auto clear_ovf = [&](int tplane) {
    float* o = &ovf[tplane & 1][0][0];
    for (int i = threadIdx.x; i < 3 * ENT; i += ENT) o[i] = 0.0f;
  };
  // cells of the staged sources of plane p
  auto cells_of = [&](int p, const float (&vu)[2][3], const float (&vg)[2][3], Src2 (&S)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      S[j].key = 0;
      S[j].t0 = S[j].t1 = S[j].t2 = 0.0f;
      S[j].g0 = vg[j][0];
      S[j].g1 = vg[j][1];
      S[j].g2 = vg[j][2];
      if (puse[j]) {
        float u0 = vu[j][0], u1 = vu[j][1], u2 = vu[j][2];
        if (FIRST) {
          u0 *= scale;
          u1 *= scale;
          u2 *= scale;
        }
        const int pc = min(max(p, 0), g.d0 - 1);
        const BorderCell bc = border_cell(g, pc, py[j], px[j], u0, u1, u2);
        const int o0 = bc.i0 - pc, r1 = bc.i1 - id.oy + 2, r2 = bc.i2 - id.ox + 2;
        const bool ok = pin[j] && p >= 0 && p < g.d0 && o0 >= -2 && o0 <= 1 && r1 >= 0 &&
                        r1 + 1 < H2Y && r2 >= 0 && r2 + 1 < H2X;
        S[j].key = ok ? (r2 | (r1 << 6) | ((o0 + 2) << 10) | (static_cast<int>(bc.k0) << 12) |
                         (static_cast<int>(bc.k1) << 13) | (static_cast<int>(bc.k2) << 14) |
                         kSrcValid)
                      : 0;
        S[j].t0 = bc.t0;
        S[j].t1 = bc.t1;
        S[j].t2 = bc.t2;
      }
    }
  };
  // bin source s of plane p if its cell lies in cell plane cz and in the
  // column's cell region
  auto bin_one = [&](int cz, int p, const Src2& sv) {
    if (!(sv.key & kSrcValid)) return;
    if (p + ((sv.key >> 10) & 3) - 2 != cz) return;
    const int cy = ((sv.key >> 6) & 15) - 1, cx = (sv.key & 63) - 1;
    if (cy < 0 || cy >= MCY || cx < 0 || cx >= MCX) return;
    const int ci = cy * MCX + cx;
    const int slot = atomicAdd(&bcnt[ci], 1);
    if (slot < KSLOT) {
      bd4[slot][ci] = make_float4(sv.t0, sv.t1, sv.t2, sv.g0);
      bd2[slot][ci] = make_float2(sv.g1, sv.g2);
    } else {
      const float w0[2] = {1.0f - sv.t0, sv.t0};
      const float w1[2] = {1.0f - sv.t1, sv.t1};
      const float w2[2] = {1.0f - sv.t2, sv.t2};
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int tz = cz + a;  // target plane
        if (tz < id.z0 || tz >= id.z1) continue;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
          for (int ee = 0; ee < 2; ++ee) {
            const int ty = cy + b - 1, tx = cx + ee - 1;
            if (ty >= 0 && ty < ETY && tx >= 0 && tx < ETX) {
              const float w = w0[a] * w1[b] * w2[ee];
              float* ov = &ovf[tz & 1][0][0] + ty * ETX + tx;
              atomicAdd(ov, w * sv.g0);
              atomicAdd(ov + ENT, w * sv.g1);
              atomicAdd(ov + 2 * ENT, w * sv.g2);
            }
          }
        }
      }
    }
  };
  // one pass over the live cell plane serves the targets of planes z and z + 1
  auto gather = [&](float (&lo)[3], float (&up)[3], bool upper) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int ci = (ly + 1 - b) * MCX + (lx + 1 - e);
#pragma unroll
        for (int j = 0; j < KSLOT; ++j) {
          const float4 q4 = bd4[j][ci];
          const float2 q2 = bd2[j][ci];
          const float w1 = b ? q4.y : 1.0f - q4.y;
          const float w12 = e ? w1 * q4.z : fmaf(-w1, q4.z, w1);
          const float wl = fmaf(-w12, q4.x, w12);
          lo[0] += wl * q4.w;
          lo[1] += wl * q2.x;
          lo[2] += wl * q2.y;
          if (upper) {
            const float wu = w12 * q4.x;
            up[0] += wu * q4.w;
            up[1] += wu * q2.x;
            up[2] += wu * q2.y;
          }
        }
      }
    }
  };

  const bool colv = pin[0];
  Src2 R0[2], R1[2], R2[2], R3[2];  // sources of four consecutive planes
  float accA[3] = {0.0f, 0.0f, 0.0f}, accB[3] = {0.0f, 0.0f, 0.0f};

  // prologue: planes z0-2 .. z0+1 staged with their cells (in R3, R0, R1,
  // R2), cell plane z0-1 filled, its a = 1 part of the plane-z0 targets;
  // plane z0+2 in flight
  clear_cells();
  clear_ovf(id.z0);
  load_plane(id.z0 - 2, pu, pg);
  store_u(id.z0 - 2, pu);
  cells_of(id.z0 - 2, pu, pg, R3);
  load_plane(id.z0 - 1, pu, pg);
  store_u(id.z0 - 1, pu);
  cells_of(id.z0 - 1, pu, pg, R0);
  load_plane(id.z0, pu, pg);
  store_u(id.z0, pu);
  cells_of(id.z0, pu, pg, R1);
  load_plane(id.z0 + 1, pu, pg);
  store_u(id.z0 + 1, pu);
  cells_of(id.z0 + 1, pu, pg, R2);
  load_plane(id.z0 + 2, pu, pg);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    bin_one(id.z0 - 1, id.z0 - 2, R3[j]);
    bin_one(id.z0 - 1, id.z0 - 1, R0[j]);
    bin_one(id.z0 - 1, id.z0, R1[j]);
    bin_one(id.z0 - 1, id.z0 + 1, R2[j]);
  }
  __syncthreads();
  {
    float none[3] = {0.0f, 0.0f, 0.0f};
    if (colv) gather(none, accA, true);
  }
  __syncthreads();

  // one plane: Sm (plane z-1), S0 (z), S1 (z+1) hold their sources, Sn
  // receives plane z+2's; (xu, xg) holds plane z+2 on entry and takes z+3;
  // acc holds the plane-z targets' a = 1 part and nacc receives plane z+1's
  auto step = [&](int z, Src2 (&Sm)[2], Src2 (&S0)[2], Src2 (&S1)[2], Src2 (&Sn)[2],
                  float (&xu)[2][3], float (&xg)[2][3], float (&acc)[3], float (&nacc)[3]) {
    // (i)
    clear_cells();
    clear_ovf(z + 1);
    store_u(z + 2, xu);
    cells_of(z + 2, xu, xg, Sn);
    load_plane(z + 3, xu, xg);
    __syncthreads();
    // (ii)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bin_one(z, z - 1, Sm[j]);
      bin_one(z, z, S0[j]);
      bin_one(z, z + 1, S1[j]);
      bin_one(z, z + 2, Sn[j]);
    }
    // (iii) direct term of the plane-z targets: the own source's cell
    float r[3] = {acc[0], acc[1], acc[2]};
    if (colv) {
      const Src2& sv = S0[0];
      Tri t;
      bool k0, k1, k2;
      if (sv.key & kSrcValid) {
        const int i0 = z + ((sv.key >> 10) & 3) - 2;
        const int sa = (i0 + 10) % 5, sb = (i0 + 11) % 5;
        const int pb = ((sv.key >> 6) & 15) * H2X + (sv.key & 63);
        float h[8];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float gcv = c == 0 ? sv.g0 : (c == 1 ? sv.g1 : sv.g2);
          const float cv[8] = {uring[sa][c][pb],       uring[sa][c][pb + 1],
                               uring[sa][c][pb + H2X], uring[sa][c][pb + H2X + 1],
                               uring[sb][c][pb],       uring[sb][c][pb + 1],
                               uring[sb][c][pb + H2X], uring[sb][c][pb + H2X + 1]};
#pragma unroll
          for (int k = 0; k < 8; ++k) h[k] = c == 0 ? gcv * cv[k] : h[k] + gcv * cv[k];
        }
        t = tri_eval(h, sv.t0, sv.t1, sv.t2);
        k0 = (sv.key >> 12) & 1;
        k1 = (sv.key >> 13) & 1;
        k2 = (sv.key >> 14) & 1;
      } else {
        // a cell outside the staged planes (not reached while every offset
        // lies in [-2, 1]): corners from memory
        float u0 = uring[(z + 10) % 5][0][pe[0]], u1 = uring[(z + 10) % 5][1][pe[0]],
              u2 = uring[(z + 10) % 5][2][pe[0]];
        if (FIRST) {
          u0 *= scale;
          u1 *= scale;
          u2 *= scale;
        }
        const BorderCell bc = border_cell(g, z, py[0], px[0], u0, u1, u2);
        t.v = 0.0f;
        t.d0 = t.d1 = t.d2 = 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float gcv = c == 0 ? sv.g0 : (c == 1 ? sv.g1 : sv.g2);
          float cv[8];
          corners_border(fc[c], g, bc.base, cv);
          const Tri tc = tri_eval(cv, bc.t0, bc.t1, bc.t2);
          t.d0 += tc.d0 * gcv;
          t.d1 += tc.d1 * gcv;
          t.d2 += tc.d2 * gcv;
        }
        k0 = bc.k0;
        k1 = bc.k1;
        k2 = bc.k2;
      }
      r[0] += sv.g0 + (k0 ? 0.0f : t.d0 * js);
      r[1] += sv.g1 + (k1 ? 0.0f : t.d1 * js);
      r[2] += sv.g2 + (k2 ? 0.0f : t.d2 * js);
    }
    __syncthreads();
    // (iv)
#pragma unroll
    for (int c = 0; c < 3; ++c) nacc[c] = 0.0f;
    if (colv) {
      gather(r, nacc, z + 1 < id.z1);
      const float* ov = &ovf[z & 1][0][0];
      r[0] += ov[threadIdx.x];
      r[1] += ov[ENT + threadIdx.x];
      r[2] += ov[2 * ENT + threadIdx.x];
      const uint32_t lin = static_cast<uint32_t>(z * g.plane + py[0] * g.d2 + px[0]);
      st_at(go, lin, r[0] * oscale);
      st_at(go + g.V, lin, r[1] * oscale);
      st_at(go + 2 * static_cast<size_t>(g.V), lin, r[2] * oscale);
    }
    __syncthreads();
  };
  // unrolled by four so that the source sets and partials keep their
  // registers
  for (int z = id.z0; z < id.z1; z += 4) {
    step(z, R0, R1, R2, R3, pu, pg, accA, accB);
    if (z + 1 < id.z1) step(z + 1, R1, R2, R3, R0, pu, pg, accB, accA);
    if (z + 2 < id.z1) step(z + 2, R2, R3, R0, R1, pu, pg, accA, accB);
    if (z + 3 < id.z1) step(z + 3, R3, R0, R1, R2, pu, pg, accB, accA);
  }
}  // the last step's barrier lets the next chunk reuse the LDS

// The subjects that the reach-1 adjoint does not take, in one launch (an idle
// launch costs as much as a small step): the first half of the blocks walks the
// column chunks of subjects with reach 2, and of those with reach 1 that the
// reach-1 adjoint left or whose gradient is not finite (the cell bins carry any
// gradient to the eight corners of its cell only); the second half the tiles of
// those with a cell offset beyond [-2, 1].  The reach alone separates the two,
// so that no subject is written by both.  Both halves step through the work
// together, block b taking items b, b + half, ..., so that the items in flight
// are neighbours (those of one XCD a contiguous range) and every block has a
// share of each subject.
__device__ __forceinline__ bool takes_far(const int* rc, bool tiled) {
  const int mr = max_reach(rc);
  return tiled ? mr > 2 : mr == 2 || (mr < 2 && (rc[kNonFinite] || rc[kFar]));
}

union FarLds {
  March2Lds march2;
  TiledBwdLds tiled;
};

template <bool FIRST>
__global__ __launch_bounds__(ENT, 3) void k_exp_bwd_far(const float* __restrict__ ut,
                                                        const float* __restrict__ gin,
                                                        float* __restrict__ gout, MarchGeom m,
                                                        BwdGeom bg, float scale, float oscale,
                                                        const int* __restrict__ boxes,
                                                        const int* __restrict__ reach) {
  __shared__ __align__(16) unsigned char lds[sizeof(FarLds)];
  FarLds& L = *reinterpret_cast<FarLds*>(lds);
  const uint32_t half = gridDim.x / 2;
  const bool tiled = blockIdx.x >= half;
  {
    // nothing to do unless some subject of the launch is this half's
    const int nsub = static_cast<int>(bg.total / bg.ntiles);
    int any = 0;
    for (int q = threadIdx.x; q < nsub; q += ENT) {
      any |= takes_far(reach + q * 8, tiled);
    }
    if (!__syncthreads_or(any)) return;
  }
  if (tiled) {
    for (uint32_t b = xcd_remap(blockIdx.x - half, half); b < bg.total; b += half) {
      const int s = static_cast<int>(b / bg.ntiles);
      if (takes_far(reach + s * 8, true))
        exp_bwd_tile<FIRST>(L.tiled, s, static_cast<int>(b - static_cast<uint32_t>(s) * bg.ntiles),
                            ut, gin, gout, bg, scale, oscale, boxes, reach);
    }
  } else {
    for (uint32_t b = xcd_remap(blockIdx.x, half); b < m.total; b += half) {
      const MarchId id = march_id_at(m, b);
      if (takes_far(reach + id.s * 8, false))
        exp_bwd_march2<FIRST>(L.march2, m, id, ut, gin, gout, scale, oscale);
    }
  }
}

// Blocks of a launch of k_exp_bwd_far: for each half as many as are resident at
// once on the current device.
template <bool FIRST>
uint32_t far_grid(uint32_t items) {
  static int cap[64] = {};
  int dev = 0;
  uint32_t half = 768u;  // when the occupancy query fails
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64) {
    int& c = cap[dev];
    if (c == 0) {
      int per_cu = 0, cus = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_exp_bwd_far<FIRST>, ENT, 0) ==
              hipSuccess &&
          hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
        c = per_cu * cus;
    }
    if (c > 0) half = static_cast<uint32_t>(c);
  }
  return 2u * (items < half ? items : half);
}

BwdGeom make_bwd(const TileGeom& tg, int n) {
  BwdGeom b;
  b.src = tg;
  b.ntx = (tg.g.d2 + BTX - 1) / BTX;
  b.nty = (tg.g.d1 + BTY - 1) / BTY;
  b.ntz = (tg.g.d0 + BTZ - 1) / BTZ;
  b.ntiles = b.ntx * b.nty * b.ntz;
  b.total = static_cast<uint32_t>(b.ntiles) * n;
  return b;
}

struct AuxPtrs {
  int* boxes;  // [n_sq][n][ntiles][8]
  int* reach;  // [n_sq][n][8]
  size_t box_stride, reach_stride;
};

AuxPtrs aux_ptrs(int* aux, const TileGeom& tg, int n, int n_sq) {
  AuxPtrs a;
  a.box_stride = static_cast<size_t>(n) * tg.ntiles * 8;
  a.reach_stride = static_cast<size_t>(n) * 8;
  a.boxes = aux;
  a.reach = aux ? aux + a.box_stride * n_sq : nullptr;
  return a;
}


// ---------------------------------------------------------------------------
// One inner iteration in one launch (small cohorts).
//
// For small volumes the marching kernels are bound by their serial planes
// (a 32^3 subject gives a squaring launch only 64 blocks of 8+ planes each)
// and by the ~20 launches of an iteration, not by memory.  This persistent
// kernel runs the whole iteration -- the squaring steps, warp + MSE/L1 +
// regulariser with their adjoints, the squaring adjoint and Adam -- as
// phases of tile-parallel work separated by grid barriers.  Its squaring
// steps gather directly (no plane ring) and write the same per-tile records
// as the marching forward; its adjoint is the tiled adjoint for every
// subject; the loss and the Adam update are the bodies of the separate
// kernels.

// One plane of a record tile (32 x 8 voxels, one per thread) of a squaring
// step: the arithmetic of k_exp_fwd<FIRST, REC> with the corners read from
// memory.  With REC the block merges cell offsets beyond [-1, 0] into the
// tile's record (which starts at that range) and the subject's reaches, which
// count from 2 on: the atomics of every plane into its tile's record took as
// long as the step itself (6.1 against 3.8 us at 4 x 32^3).  Blocks are
// (subject, tile, plane), so a small volume gets eight times the blocks of the
// marching kernel and no serial planes.
template <bool FIRST, bool REC>
__device__ __forceinline__ void exp_fwd_plane_body(int (*red)[ENT / 64], uint32_t blk,
                                                   const float* __restrict__ src,
                                                   float* __restrict__ dst, const TileGeom& tg,
                                                   float scale, int* __restrict__ boxes,
                                                   int* __restrict__ reach) {
  const Geom& g = tg.g;
  const uint32_t b = xcd_remap(blk, tg.total * ETZ);
  const uint32_t bt = b / ETZ;
  const int k = static_cast<int>(b - bt * ETZ);
  const int s = static_cast<int>(bt / tg.ntiles);
  const int tile = static_cast<int>(bt - static_cast<uint32_t>(s) * tg.ntiles);
  const int ox = (tile % tg.ntx) * ETX;
  const int oy = ((tile / tg.ntx) % tg.nty) * ETY;
  const int x0 = (tile / (tg.ntx * tg.nty)) * ETZ + k;
  const size_t off = static_cast<size_t>(s) * 3 * g.V;
  const float* f = src + off;
  float* o = dst + off;
  const float* fc[3] = {f, f + g.V, f + 2 * static_cast<size_t>(g.V)};
  const int lx = threadIdx.x % ETX, ly = threadIdx.x / ETX;
  const int x2 = ox + lx, x1 = oy + ly;
  int mn0 = INT_MAX, mn1 = INT_MAX, mn2 = INT_MAX, mx0 = INT_MIN, mx1 = INT_MIN, mx2 = INT_MIN;
  if (x2 < g.d2 && x1 < g.d1 && x0 < g.d0) {
    const uint32_t lin = static_cast<uint32_t>(x0 * g.plane + x1 * g.d2 + x2);
    float u0 = ld_at(fc[0], lin), u1 = ld_at(fc[1], lin), u2 = ld_at(fc[2], lin);
    if (FIRST) {
      u0 *= scale;
      u1 *= scale;
      u2 *= scale;
    }
    const BorderCell bc = border_cell(g, x0, x1, x2, u0, u1, u2);
    float cv[3][8];
#pragma unroll
    for (int c = 0; c < 3; ++c) corners_border(fc[c], g, bc.base, cv[c]);
    float r[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r[c] = tri_value(cv[c], bc.t0, bc.t1, bc.t2);
      if (FIRST) r[c] *= scale;
    }
    st_at(o, lin, u0 + r[0]);
    st_at(o + g.V, lin, u1 + r[1]);
    st_at(o + 2 * static_cast<size_t>(g.V), lin, u2 + r[2]);
    mn0 = mx0 = bc.i0 - x0;
    mn1 = mx1 = bc.i1 - x1;
    mn2 = mx2 = bc.i2 - x2;
  }
  if (REC) {
    mn0 = wave_min(mn0);
    mn1 = wave_min(mn1);
    mn2 = wave_min(mn2);
    mx0 = wave_max(mx0);
    mx1 = wave_max(mx1);
    mx2 = wave_max(mx2);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) {
      red[0][w] = mn0;
      red[1][w] = mn1;
      red[2][w] = mn2;
      red[3][w] = mx0;
      red[4][w] = mx1;
      red[5][w] = mx2;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
      const int q = threadIdx.x;
      int r = red[q][0];
      for (int i = 1; i < ENT / 64; ++i) r = q < 3 ? min(r, red[q][i]) : max(r, red[q][i]);
      int* bx = boxes + (static_cast<size_t>(s) * tg.ntiles + tile) * 8;
      if (q < 3 && r < -1) {
        atomicMin(bx + q, r);
        atomicMax(reach + s * 8 + q, -r);
      } else if (q >= 3 && r > 0) {
        atomicMax(bx + q, r);
        atomicMax(reach + s * 8 + q, r + 1);
      }
    }
    __syncthreads();  // `red` is rewritten by the block's next plane
  }
}

// Value that entry e of a record box starts at before planes merge into it:
// offsets in [-1, 0].
__device__ __forceinline__ int box_start(int e) { return e < 3 ? -1 : 0; }

// Boxes of `nbox` entries, followed by nreach zeroed reaches.
__global__ __launch_bounds__(ENT) void k_aux_init(int* __restrict__ aux, long long nbox,
                                                  long long nreach) {
  const long long stride = static_cast<long long>(gridDim.x) * ENT;
  for (long long i = static_cast<long long>(blockIdx.x) * ENT + threadIdx.x; i < nbox + nreach;
       i += stride)
    aux[i] = i < nbox ? box_start(static_cast<int>(i & 7)) : 0;
}

template <bool FIRST, bool REC>
__global__ __launch_bounds__(ENT) void k_exp_fwd_planes(const float* __restrict__ src,
                                                        float* __restrict__ dst, TileGeom tg,
                                                        float scale, int* __restrict__ boxes,
                                                        int* __restrict__ reach) {
  __shared__ int red[6][ENT / 64];
  exp_fwd_plane_body<FIRST, REC>(red, blockIdx.x, src, dst, tg, scale, boxes, reach);
}

// Grid-wide barrier of a launch whose blocks are all resident.  bar[0]
// counts arrivals over the launch (zeroed before it); the k-th barrier
// returns once k * gridDim.x blocks have arrived.  The wait is bounded by the
// real-time counter: a block that has waited `ticks` raises err[0] and goes
// on, so every wave reaches the end of the kernel even if some block never
// ran.
__device__ __forceinline__ void grid_barrier(unsigned* bar, int* err, unsigned k,
                                             long long ticks) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    atomicAdd(bar, 1u);
    const unsigned target = k * gridDim.x;
    const long long t0 = wall_clock64();
    while (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (wall_clock64() - t0 > ticks) {
        atomicOr(err, 1);
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    __threadfence();
  }
  __syncthreads();
}

struct IterArgs {
  const float* img;    // [B][V]
  const float* atlas;  // [V]
  float* v;            // [B][3][V], updated in place (no smoothing on this path)
  float* m;
  float* s;
  float* v_out;        // Adam's outputs: v, m, s themselves, or scratch when timing
  float* m_out;
  float* s_out;
  float* ckpt;         // [n_sq - 1][B][3][V]
  float* uN;
  float* gU;
  float* gA;
  float* gB;
  float* gV;
  int* boxes;          // [n_sq][B][ntiles][8]
  int* reach;          // [n_sq][B][8]
  size_t box_stride, reach_stride;
  double* loss;        // loss[b * loss_stride] += L_b
  int loss_stride;
  RegW rw;
  TileGeom tg;
  BwdGeom bg;
  int n_sq;
  float scale;         // 2^-n_sq
  double inv_v;
  uint32_t nbx;        // voxel blocks per subject
  long long count;     // B * 3V
  const long long* step_dev;  // device step count, or NULL: step_host
  long long step_host;
  int k;               // inner iteration within the sweep
  float lr;
  double b1, b2;
  float eps;
  unsigned* bar;
  int* err;
  long long ticks;     // bound of a barrier wait (real-time counter ticks)
};

constexpr size_t kIterLds = sizeof(TiledBwdLds);

template <bool L1>
__global__ __launch_bounds__(ENT) void k_iter_fused(IterArgs a) {
  __shared__ __align__(16) unsigned char lds[kIterLds];
  const Geom& g = a.tg.g;
  const uint32_t G = gridDim.x;
  const size_t fs = static_cast<size_t>(a.tg.total / a.tg.ntiles) * 3 * g.V;
  unsigned nbar = 0;
  // the records are running minima / maxima: start the reaches at zero and
  // the boxes at offsets [-1, 0]
  {
    const long long cnt = static_cast<long long>(a.reach_stride) * a.n_sq;
    for (long long i = static_cast<long long>(blockIdx.x) * ENT + threadIdx.x; i < cnt;
         i += static_cast<long long>(G) * ENT)
      a.reach[i] = 0;
    const long long nb = static_cast<long long>(a.box_stride) * a.n_sq;
    for (long long i = static_cast<long long>(blockIdx.x) * ENT + threadIdx.x; i < nb;
         i += static_cast<long long>(G) * ENT) {
      a.boxes[i] = box_start(static_cast<int>(i & 7));
    }
  }
  grid_barrier(a.bar, a.err, ++nbar, a.ticks);
  // squaring steps (u_0 = v / 2^N scaled on the fly), records for the adjoint
  int (*red)[ENT / 64] = reinterpret_cast<int(*)[ENT / 64]>(lds);
  const float* src = a.v;
  for (int t = 0; t < a.n_sq; ++t) {
    float* dst = (t == a.n_sq - 1) ? a.uN : a.ckpt + static_cast<size_t>(t) * fs;
    int* bx = a.boxes + a.box_stride * t;
    int* rc = a.reach + a.reach_stride * t;
    for (uint32_t b = blockIdx.x; b < a.tg.total * ETZ; b += G) {
      if (t == 0)
        exp_fwd_plane_body<true, true>(red, b, src, dst, a.tg, a.scale, bx, rc);
      else
        exp_fwd_plane_body<false, true>(red, b, src, dst, a.tg, 1.0f, bx, rc);
    }
    grid_barrier(a.bar, a.err, ++nbar, a.ticks);
    src = dst;
  }
  // dissimilarity + regulariser, and dL/du_N
  {
    const uint32_t total = a.nbx * (a.tg.total / a.tg.ntiles);
    double* rd = reinterpret_cast<double*>(lds);
    for (uint32_t b = blockIdx.x; b < total; b += G)
      mse_fused_block<L1, true>(xcd_remap(b, total), rd, a.img, a.atlas, a.uN, a.gU, a.loss,
                                a.loss_stride, a.rw, g, a.inv_v, a.nbx);
  }
  grid_barrier(a.bar, a.err, ++nbar, a.ticks);
  // squaring adjoint, every subject on the tiled path
  TiledBwdLds& L = *reinterpret_cast<TiledBwdLds*>(lds);
  const float* gin = a.gU;
  for (int t = a.n_sq - 1; t >= 0; --t) {
    float* gout = (t == 0) ? a.gV : (((a.n_sq - 1 - t) % 2 == 0) ? a.gA : a.gB);
    const float* ut = (t == 0) ? a.v : a.ckpt + static_cast<size_t>(t - 1) * fs;
    const int* bx = a.boxes + a.box_stride * t;
    const int* rc = a.reach + a.reach_stride * t;
    for (uint32_t b = blockIdx.x; b < a.bg.total; b += G) {
      const uint32_t bid = xcd_remap(b, a.bg.total);
      const int sub = static_cast<int>(bid / a.bg.ntiles);
      const int tile = static_cast<int>(bid - static_cast<uint32_t>(sub) * a.bg.ntiles);
      if (t == 0)
        exp_bwd_tile<true>(L, sub, tile, ut, gin, gout, a.bg, a.scale, a.scale, bx, rc);
      else
        exp_bwd_tile<false>(L, sub, tile, ut, gin, gout, a.bg, 1.0f, 1.0f, bx, rc);
    }
    grid_barrier(a.bar, a.err, ++nbar, a.ticks);
    gin = gout;
  }
  // Adam; bias corrections formed in FP64 and rounded once, as the separate
  // kernels do
  const double tt = static_cast<double>((a.step_dev ? a.step_dev[0] : a.step_host) + a.k + 1);
  const float bc1 = static_cast<float>(1.0 - pow(a.b1, tt));
  const float bc2 = static_cast<float>(1.0 - pow(a.b2, tt));
  const float b1f = static_cast<float>(a.b1), b2f = static_cast<float>(a.b2);
  const float omb1 = static_cast<float>(1.0 - a.b1), omb2 = static_cast<float>(1.0 - a.b2);
  for (long long i = static_cast<long long>(blockIdx.x) * ENT + threadIdx.x; i < a.count;
       i += static_cast<long long>(G) * ENT)
    adam_step_to(a.v, a.m, a.s, a.gV, a.v_out, a.m_out, a.s_out, i, a.lr, b1f, omb1, b2f, omb2,
                 bc1, bc2, a.eps);
}

// A barrier that timed out leaves NaN as the group loss.
__global__ void k_flag_loss(const int* __restrict__ err, double* __restrict__ out) {
  if (threadIdx.x == 0 && blockIdx.x == 0 && err[0]) out[0] = __builtin_nan("");
}
}  // namespace

size_t exp_aux_bytes(const Geom& g, int n, int n_sq) {
  const TileGeom tg = make_tiles(g, n);
  return (static_cast<size_t>(n) * tg.ntiles * 8 + static_cast<size_t>(n) * 8) * n_sq *
         sizeof(int);
}

// Chunk length along d0 of the marching kernels.
int march_tz(const TileGeom& tg, int n) {
  const int tuned = tuned_tz(TUNE_EXP, tg.g, n);
  if (tuned > 1) return tuned;
  if (tuned < 0) return ETZ;  // plane-parallel kernels; the chunk is not used
  // long chunks amortise the ramp-up planes, short ones keep each block's
  // planes in flight within L2 (64 planes measured no faster than 32 and
  // fetched more from HBM); shorter still until there are 4096 columns of 8 rows
  // (2048 of 16): seven adjoint steps of 4 x 160 x 192 x 160 in chunks of 8, 16 and
  // 32 planes 1.60, 1.57 and 1.77 ms (taken: 16), 8 x 96^3 641, 635 and 806 us
  // (8), 4 x 128^3 718, 679 and 819 (8), 4 x 96 x 112 x 96 383, 450 and 644 (8)
  int tz = 32;
  while (tz > ETZ && static_cast<long long>(tg.ntx) * tg.nty * ((tg.g.d0 + tz - 1) / tz) * n < 4096)
    tz /= 2;
  return tz;
}

// The other shape of the squaring steps and their adjoint: one plane of a
// tile per block (k_exp_fwd_planes) and an adjoint tile per block
// (k_exp_bwd_small), no marching.  It wins on small volumes, where the marching kernels' serial
// planes are the whole cost (4 x 32^3: half the time per sweep).
// Untuned, it is taken where 8-plane chunks make fewer than 1024 columns of 8
// rows (about 512 of the adjoint's 16), where the adjoint is even: seven steps and
// seven adjoints of 4 x 64^3 (512) 83 and 164 us, marching 73 and 220; 4 x 72^3
// (972) 122 and 269, 94 and 275; 4 x 80^3 (1200) 144 and 310, 107 and 292.
bool plane_mode(const Geom& g, int n) {
  const int tuned = tuned_tz(TUNE_EXP, g, n);
  if (tuned != 0) return tuned < 0;
  const long long march_blocks = static_cast<long long>((g.d2 + ETX - 1) / ETX) *
                                 ((g.d1 + ETY - 1) / ETY) * ((g.d0 + ETZ - 1) / ETZ) * n;
  return march_blocks < 1024;
}

namespace {

// One marching squaring step (records when bx is given).
template <bool FIRST, bool REC, int ROWS>
void launch_exp_fwd_r(const float* src, float* dst, const HatGeom& hg, const TileGeom& tg,
                      float scale, int* bx, int* rc, hipStream_t st) {
  if (streamed(dst, static_cast<size_t>(tg.total / tg.ntiles) * 3 * tg.g.V, tg.g))
    hipLaunchKernelGGL((k_exp_fwd<FIRST, REC, true, ROWS>), dim3(hg.total), dim3(ENT), 0, st, src,
                       dst, hg, tg, scale, bx, rc);
  else
    hipLaunchKernelGGL((k_exp_fwd<FIRST, REC, false, ROWS>), dim3(hg.total), dim3(ENT), 0, st, src,
                       dst, hg, tg, scale, bx, rc);
}

// Columns of 16 rows fetch less halo; of 8, there are twice as many and fewer
// idle rows.  16 where that makes six blocks per CU, adds at most a fifth to the
// rows, and rows are whole 64-byte pieces (or most of one column).  Seven steps
// in columns of 8 and 16: 16 x 160 x 192 x 160 (6000 blocks of 16 rows) 3.11 and
// 2.88 ms, 8 x 96^3 (1728) 318 and 305 us; 2 x 128^3 (1024) 172 and 178, 4 x 80^3
// (600) 107 and 120; 8 x 128 x 24 x 128 129 and 151; 16 x 182 x 218 x 182 6.02 and
// 6.42 ms; 8 x 256 x 256 x 24 616 and 566 us.
template <bool FIRST, bool REC>
void launch_exp_fwd_c(const float* src, float* dst, const TileGeom& tg, int tz, float scale,
                      int* bx, int* rc, hipStream_t st) {
  const HatGeom wide = make_hat(tg, tz, Column<2>::TY), one = make_hat(tg, tz, Column<1>::TY);
  const bool rows = 5 * Column<2>::TY * wide.nty <= 6 * Column<1>::TY * one.nty;
  const bool whole = tg.g.d2 % 16 == 0 || (tg.g.d2 > ETX / 2 && tg.g.d2 < ETX);
  if (wide.total >= 1536 && rows && whole)
    launch_exp_fwd_r<FIRST, REC, 2>(src, dst, wide, tg, scale, bx, rc, st);
  else
    launch_exp_fwd_r<FIRST, REC, 1>(src, dst, one, tg, scale, bx, rc, st);
}

void launch_exp_fwd(const float* src, float* dst, bool first, const TileGeom& tg, int tz,
                    float scale, int* bx, int* rc, hipStream_t st) {
  if (first && bx)
    launch_exp_fwd_c<true, true>(src, dst, tg, tz, scale, bx, rc, st);
  else if (first)
    launch_exp_fwd_c<true, false>(src, dst, tg, tz, scale, bx, rc, st);
  else if (bx)
    launch_exp_fwd_c<false, true>(src, dst, tg, tz, scale, bx, rc, st);
  else
    launch_exp_fwd_c<false, false>(src, dst, tg, tz, scale, bx, rc, st);
}

// One squaring step in the launch's shape.
void launch_fwd_step(const float* src, float* dst, bool first, bool planes, const TileGeom& tg,
                     int tz, float scale, int* bx, int* rc, hipStream_t st) {
  if (!planes) return launch_exp_fwd(src, dst, first, tg, tz, scale, bx, rc, st);
  const dim3 grid(tg.total * ETZ);
  if (first && bx)
    hipLaunchKernelGGL((k_exp_fwd_planes<true, true>), grid, dim3(ENT), 0, st, src, dst, tg, scale,
                       bx, rc);
  else if (first)
    hipLaunchKernelGGL((k_exp_fwd_planes<true, false>), grid, dim3(ENT), 0, st, src, dst, tg, scale,
                       bx, rc);
  else if (bx)
    hipLaunchKernelGGL((k_exp_fwd_planes<false, true>), grid, dim3(ENT), 0, st, src, dst, tg, scale,
                       bx, rc);
  else
    hipLaunchKernelGGL((k_exp_fwd_planes<false, false>), grid, dim3(ENT), 0, st, src, dst, tg,
                       scale, bx, rc);
}

// The reach-1 adjoint of one step (check: no records were taken).
template <bool FIRST, bool CHECK>
void launch_hat_r(const float* ut, const float* gin, float* gout, const HatGeom& hg, int n,
                  float scale, int* rc, const int* later, hipStream_t st) {
  if (streamed(gout, static_cast<size_t>(n) * 3 * hg.g.V, hg.g))
    hipLaunchKernelGGL((k_exp_bwd_hat<FIRST, CHECK, true>), dim3(hg.total), dim3(ENT), 0, st, ut,
                       gin, gout, hg, scale, scale, rc, later);
  else
    hipLaunchKernelGGL((k_exp_bwd_hat<FIRST, CHECK, false>), dim3(hg.total), dim3(ENT), 0, st, ut,
                       gin, gout, hg, scale, scale, rc, later);
}

}  // namespace

void run_exp_fwd(const float* v, float* u, float* ckpt, float* tmp, int* aux, const Geom& g, int n,
                 int n_sq, hipStream_t st, bool negate) {
  const size_t fs = static_cast<size_t>(n) * 3 * g.V;
  if (n_sq == 0) {
    prof_begin(st, KC_MISC);
    (void)hipMemcpyAsync(u, v, fs * sizeof(float), hipMemcpyDeviceToDevice, st);
    prof_end(st, KC_MISC);
    return;
  }
  const TileGeom tg = make_tiles(g, n);
  const int tz = march_tz(tg, n);
  const AuxPtrs ap = aux_ptrs(aux, tg, n, n_sq);
  const bool planes = plane_mode(g, n);
  // the reaches are running maxima: start them at zero (all-zero bits); the
  // planes kernel merges into its boxes too
  if (aux && planes) {
    const long long nbox = static_cast<long long>(ap.box_stride) * n_sq;
    const long long nreach = static_cast<long long>(ap.reach_stride) * n_sq;
    prof_begin(st, KC_FILL);
    hipLaunchKernelGGL(k_aux_init, dim3(static_cast<uint32_t>(
                                       (nbox + nreach) / ENT + 1 < 65536 ? (nbox + nreach) / ENT + 1
                                                                         : 65536)),
                       dim3(ENT), 0, st, aux, nbox, nreach);
    prof_end(st, KC_FILL);
  } else if (aux) {
    launch_fill_f32(reinterpret_cast<float*>(ap.reach),
                    static_cast<long long>(ap.reach_stride) * n_sq, 0.0f, st);
  }
  // Exp(-v) negates the scaled field of the first step (exact)
  const float scale = negate ? -ldexpf(1.0f, -n_sq) : ldexpf(1.0f, -n_sq);
  const float* src = v;
  for (int t = 0; t < n_sq; ++t) {
    float* dst;
    if (t == n_sq - 1)
      dst = u;
    else if (ckpt)
      dst = ckpt + static_cast<size_t>(t) * fs;  // slot t holds u_{t+1}
    else
      dst = ((n_sq - 1 - t) % 2 == 0) ? u : tmp;  // ping-pong ending in u
    int* bx = aux ? ap.boxes + ap.box_stride * t : nullptr;
    int* rc = aux ? ap.reach + ap.reach_stride * t : nullptr;
    prof_begin(st, KC_EXP_FWD);
    launch_fwd_step(src, dst, t == 0, planes, tg, tz, t == 0 ? scale : 1.0f, bx, rc, st);
    prof_end(st, KC_EXP_FWD);
    src = dst;
  }
}

namespace {

// Records of steps t0 .. t0 + steps - 1 (of flagged subjects only).
void launch_rec(const float* v, const float* ckpt, size_t fs, int t0, int steps,
                const TileGeom& tg, float scale, const AuxPtrs& ap, bool flagged,
                hipStream_t st) {
  const uint32_t blocks = flagged && tg.total > 2048u ? 2048u : tg.total;
  prof_begin(st, KC_MISC);
  hipLaunchKernelGGL(k_exp_rec, dim3(blocks, steps), dim3(ENT), 0, st, v, ckpt, fs, t0, tg, scale,
                     ap.boxes, ap.box_stride, ap.reach, ap.reach_stride, flagged);
  prof_end(st, KC_MISC);
}

// The adjoint of step t.  recs: the records of this step were taken (always in
// the plane-parallel shape); otherwise those of the subjects that need them
// are taken here, from u_t = ut (the launch's step t of `v` and `ut`).
void launch_bwd_step(const float* ut, const float* gin, float* gout, int t, int n_sq, bool recs,
                     const MarchGeom& m, const BwdGeom& bg, float scale, const AuxPtrs& ap,
                     bool planes, hipStream_t st) {
  const bool first = t == 0;
  const float sc = first ? scale : 1.0f;
  const int* bx = ap.boxes + ap.box_stride * t;
  int* rc = ap.reach + ap.reach_stride * t;
  if (planes) {
    const NearGeom ng = make_near(bg);
    const dim3 grid(static_cast<uint32_t>(ng.items) * (bg.total / bg.ntiles));
    prof_begin(st, KC_EXP_BWD);
    if (first)
      hipLaunchKernelGGL((k_exp_bwd_small<true>), grid, dim3(ENT), 0, st, ut, gin, gout, ng, sc,
                         sc, bx, rc);
    else
      hipLaunchKernelGGL((k_exp_bwd_small<false>), grid, dim3(ENT), 0, st, ut, gin, gout, ng, sc,
                         sc, bx, rc);
    prof_end(st, KC_EXP_BWD);
    return;
  }
  // each subject's result comes from one of the three adjoints, decided on the
  // device from its reach (1, 2, beyond) and the reach-1 kernel's marks; what
  // the reach-1 kernel wrote of a subject that it left is overwritten
  const HatGeom hg = make_hat(m.rec, m.tz, HTY);
  const int* later = !recs && t + 1 < n_sq ? rc + ap.reach_stride : nullptr;
  prof_begin(st, KC_EXP_BWD);
  const int n = static_cast<int>(m.rec.total / m.rec.ntiles);
  if (first && recs)
    launch_hat_r<true, false>(ut, gin, gout, hg, n, sc, rc, later, st);
  else if (first)
    launch_hat_r<true, true>(ut, gin, gout, hg, n, sc, rc, later, st);
  else if (recs)
    launch_hat_r<false, false>(ut, gin, gout, hg, n, sc, rc, later, st);
  else
    launch_hat_r<false, true>(ut, gin, gout, hg, n, sc, rc, later, st);
  if (!recs) {
    prof_end(st, KC_EXP_BWD);
    // (the kernel takes step t > 0 from ckpt + (t - 1) fields)
    AuxPtrs one = ap;
    one.boxes = ap.boxes + ap.box_stride * t;
    one.reach = rc;
    one.box_stride = one.reach_stride = 0;
    launch_rec(ut, ut, 0, first ? 0 : 1, 1, m.rec, sc, one, true, st);
    prof_begin(st, KC_EXP_BWD);
  }
  const uint32_t items = m.total > bg.total ? m.total : bg.total;
  if (first)
    hipLaunchKernelGGL((k_exp_bwd_far<true>), dim3(far_grid<true>(items)), dim3(ENT), 0, st, ut,
                       gin, gout, m, bg, sc, sc, bx, rc);
  else
    hipLaunchKernelGGL((k_exp_bwd_far<false>), dim3(far_grid<false>(items)), dim3(ENT), 0, st, ut,
                       gin, gout, m, bg, sc, sc, bx, rc);
  prof_end(st, KC_EXP_BWD);
}

}  // namespace

void run_exp_bwd(const float* v, const float* ckpt, const float* g_u, float* g_v, float* tmp_a,
                 float* tmp_b, int* aux, bool aux_ready, const Geom& g, int n, int n_sq,
                 hipStream_t st) {
  const size_t fs = static_cast<size_t>(n) * 3 * g.V;
  if (n_sq == 0) {
    prof_begin(st, KC_MISC);
    (void)hipMemcpyAsync(g_v, g_u, fs * sizeof(float), hipMemcpyDeviceToDevice, st);
    prof_end(st, KC_MISC);
    return;
  }
  const TileGeom tg = make_tiles(g, n);
  const BwdGeom bg = make_bwd(tg, n);
  const MarchGeom m = make_march(tg, n, march_tz(tg, n));
  const AuxPtrs ap = aux_ptrs(aux, tg, n, n_sq);
  const float scale = ldexpf(1.0f, -n_sq);
  const bool planes = plane_mode(g, n);
  if (!aux_ready) {
    launch_fill_f32(reinterpret_cast<float*>(ap.reach),
                    static_cast<long long>(ap.reach_stride) * n_sq, 0.0f, st);
    // a small launch takes every step's records at once; the marching adjoint
    // looks for itself and has them taken only where it needs them (a pass over
    // u per step otherwise: 0.24 ms beside 1.17 at 16 x 160 x 192 x 224)
    if (planes) launch_rec(v, ckpt, fs, 0, n_sq, tg, scale, ap, false, st);
  }
  const float* gin = g_u;
  for (int t = n_sq - 1; t >= 0; --t) {
    float* gout = (t == 0) ? g_v : (((n_sq - 1 - t) % 2 == 0) ? tmp_a : tmp_b);
    const float* ut = (t == 0) ? v : ckpt + static_cast<size_t>(t - 1) * fs;
    launch_bwd_step(ut, gin, gout, t, n_sq, aux_ready, m, bg, scale, ap, planes, st);
    gin = gout;
  }
}

void run_exp_bwd_recompute(const float* v, const float* g_u, float* g_v, float* tmp_a,
                           float* tmp_b, float* rec_a, float* rec_b, int* aux, const Geom& g,
                           int n, int n_sq, hipStream_t st) {
  const TileGeom tg = make_tiles(g, n);
  const BwdGeom bg = make_bwd(tg, n);
  const MarchGeom m = make_march(tg, n, march_tz(tg, n));
  const AuxPtrs ap = aux_ptrs(aux, tg, n, n_sq);
  const float scale = ldexpf(1.0f, -n_sq);
  const bool planes = plane_mode(g, n);
  launch_fill_f32(reinterpret_cast<float*>(ap.reach),
                  static_cast<long long>(ap.reach_stride) * n_sq, 0.0f, st);
  const float* gin = g_u;
  for (int t = n_sq - 1; t >= 0; --t) {
    // u_t = t squaring steps of v / 2^N, ping-ponging so that it ends in rec_a
    const float* ut = v;
    for (int k = 0; k < t; ++k) {
      float* dst = ((t - 1 - k) % 2 == 0) ? rec_a : rec_b;
      prof_begin(st, KC_EXP_FWD);
      launch_fwd_step(ut, dst, k == 0, planes, tg, m.tz, k == 0 ? scale : 1.0f, nullptr, nullptr,
                      st);
      prof_end(st, KC_EXP_FWD);
      ut = dst;
    }
    // u_t stands in place of every step's field
    if (planes) launch_rec(t == 0 ? v : ut, ut, 0, t, 1, tg, scale, ap, false, st);
    float* gout = (t == 0) ? g_v : (((n_sq - 1 - t) % 2 == 0) ? tmp_a : tmp_b);
    launch_bwd_step(ut, gin, gout, t, n_sq, false, m, bg, scale, ap, planes, st);
    gin = gout;
  }
}

namespace {

long long g_barrier_ticks = kDefaultBarrierTicks;

// Resident blocks of the fused kernel on the current device (0 when the
// query fails).
template <bool L1>
int fused_capacity() {
  static int cap[2][64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int& c = cap[L1 ? 1 : 0][dev];
  if (c == 0) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_iter_fused<L1>, ENT, 0) !=
            hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return 0;
    c = per_cu * cus;
  }
  return c;
}

template <bool L1>
bool launch_iter(const IterArgs& a, uint32_t needed, hipStream_t st) {
  const int cap = fused_capacity<L1>();
  if (cap < 8) return false;
  uint32_t grid = needed < static_cast<uint32_t>(cap) ? needed : static_cast<uint32_t>(cap);
  // a multiple of the 8 XCDs, so that the XCD of a virtual block index is
  // that of the hardware block running it
  // at most 128 blocks: every block's agent-scope fence in a grid barrier
  // writes back its XCD's L2, and the fences serialise (measured 4.6 us per
  // barrier at 64 blocks, 8.1 at 128, 37 at 512)
  grid = grid < 128u ? grid : 128u;
  grid = grid >= 8 ? grid / 8 * 8 : 8;
  if (grid > static_cast<uint32_t>(cap)) return false;
  hipLaunchKernelGGL((k_iter_fused<L1>), dim3(grid), dim3(ENT), 0, st, a);
  return true;
}

}  // namespace

bool run_iter_fused(const float* img, const float* atlas, float* v, float* m, float* s,
                    float* ckpt, int* aux, float* uN, float* gU, float* gA, float* gB, float* gV,
                    double* loss, int loss_stride, const RegW& rw, const Geom& g, int n, int n_sq,
                    const long long* step_dev, long long step_host, int k, float lr, double b1,
                    double b2, float eps, bool l1, unsigned* bar, int* err, hipStream_t st,
                    float* v_out, float* m_out, float* s_out) {
  if (n_sq < 1 || (!ckpt && n_sq >= 2)) return false;
  const TileGeom tg = make_tiles(g, n);
  const AuxPtrs ap = aux_ptrs(aux, tg, n, n_sq);
  IterArgs a;
  a.img = img;
  a.atlas = atlas;
  a.v = v;
  a.m = m;
  a.s = s;
  a.v_out = v_out ? v_out : v;
  a.m_out = m_out ? m_out : m;
  a.s_out = s_out ? s_out : s;
  a.ckpt = ckpt;
  a.uN = uN;
  a.gU = gU;
  a.gA = gA;
  a.gB = gB;
  a.gV = gV;
  a.boxes = ap.boxes;
  a.reach = ap.reach;
  a.box_stride = ap.box_stride;
  a.reach_stride = ap.reach_stride;
  a.loss = loss;
  a.loss_stride = loss_stride;
  a.rw = rw;
  a.tg = tg;
  a.bg = make_bwd(tg, n);
  a.n_sq = n_sq;
  a.scale = ldexpf(1.0f, -n_sq);
  a.inv_v = 1.0 / g.V;
  a.nbx = blocks_for(g.V, kBlock);
  a.count = static_cast<long long>(n) * 3 * g.V;
  a.step_dev = step_dev;
  a.step_host = step_host;
  a.k = k;
  a.lr = lr;
  a.b1 = b1;
  a.b2 = b2;
  a.eps = eps;
  a.bar = bar;
  a.err = err;
  a.ticks = g_barrier_ticks;
  const uint32_t nv = a.nbx * static_cast<uint32_t>(n);
  uint32_t needed = tg.total * ETZ > nv ? tg.total * ETZ : nv;
  needed = needed > a.bg.total ? needed : a.bg.total;
  // the arrival counter starts every launch at zero (a fill kernel, so that
  // the sequence can be captured)
  launch_fill_f32(reinterpret_cast<float*>(bar), 1, 0.0f, st);
  prof_begin(st, KC_ITER);
  const bool ok = l1 ? launch_iter<true>(a, needed, st) : launch_iter<false>(a, needed, st);
  prof_end(st, KC_ITER);
  return ok;
}

void flag_fused_error(const int* err, double* out, hipStream_t st) {
  prof_begin(st, KC_MISC);
  hipLaunchKernelGGL(k_flag_loss, dim3(1), dim3(64), 0, st, err, out);
  prof_end(st, KC_MISC);
}

void set_barrier_ticks(long long ticks) {
  g_barrier_ticks = ticks < 0 ? kDefaultBarrierTicks : ticks;
}

int fused_resident_blocks(bool l1) { return l1 ? fused_capacity<true>() : fused_capacity<false>(); }

}  // namespace darc
