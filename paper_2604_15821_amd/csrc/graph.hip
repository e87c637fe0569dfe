// Neighbour list, reverse-edge map, edge geometry and the radial basis.
//
// Paper Sec. "MatRIS": the graph generation module repeats a structure
// periodically and connects atoms closer than the cutoff; the embedding
// module turns distances into edge features.  The inclusion rule (an fp32
// expression with a fixed operation order and no fused multiply-add), the
// canonical (i, j, n) order and the basis are the readings documented with
// janus_build_edges and in the design notes.
#include <cmath>

#include "internal.h"
#include "kernels.h"

namespace janus {

// Image half-widths m_k = floor(r_cut / L_k) + 1 of a diagonal cell.
__device__ __forceinline__ void image_range(const float* L, float rc, int& mx, int& my, int& mz) {
  mx = (int)floor((double)rc / (double)L[0]) + 1;
  my = (int)floor((double)rc / (double)L[4]) + 1;
  mz = (int)floor((double)rc / (double)L[8]) + 1;
}

// All-pairs candidates n_s * n_images from which a structure may use the cell list in mode 0.  The whole
// build at r_cut = 6 and 0.1 atoms per cubic Angstrom, all pairs against cell list in us, for 1, 4 and 16 cells:
//   27 images, 2048 atoms (55 296 candidates)  179 177, 264 301, 654 769
//   27 images, 2500 atoms (67 500)             206 190, 343 332, 887 893
//   27 images, 3000 atoms (81 000)             232 189, 438 387, 1156 1070
//   75 images,  600 atoms (45 000)             173 203, 195 234, 357 456
//   75 images,  900 atoms (67 500)             233 210, 280 264, 644 610
//   75 images, 1100 atoms (82 500)             270 212, 356 299, 863 709
// The two meet between 55 000 and 68 000 whatever the number of cells and images.
constexpr long long kCellMinCand = 65536;

// Flag bits: 1 bad offsets, 2 unsupported cell, 32 (with rc > 0) a structure that may use the cell list.
__global__ void validate_struct_kernel(const int* __restrict__ offsets, int S, int N, const float* __restrict__ cell,
                                       float rc, int* __restrict__ flag) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s > S) return;
  int bad = 0;
  if (s == 0 && offsets[0] != 0) bad |= 1;
  if (s == S && offsets[S] != N) bad |= 1;
  if (s < S) {
    if (offsets[s] > offsets[s + 1]) bad |= 1;
    if (rc > 0.f) {
      const float* L = cell + 9 * s;
      if (L[1] != 0.f || L[2] != 0.f || L[3] != 0.f || L[5] != 0.f || L[6] != 0.f || L[7] != 0.f) bad |= 2;
      if (!(L[0] > 0.f) || !(L[4] > 0.f) || !(L[8] > 0.f)) bad |= 2;
      // image shifts are stored as int8 and the candidate count must stay small
      else if ((double)rc / L[0] > 60.0 || (double)rc / L[4] > 60.0 || (double)rc / L[8] > 60.0) bad |= 2;
      else if (!(bad & 1)) {
        int mx, my, mz;
        image_range(L, rc, mx, my, mz);
        const long long nimg = (long long)(2 * mx + 1) * (2 * my + 1) * (2 * mz + 1);
        if ((long long)(offsets[s + 1] - offsets[s]) * nimg >= kCellMinCand) bad |= 32;
      }
    }
  }
  if (bad) atomicOr(flag, bad);
}

// sid[a] = structure of atom a (clamped so that bad offsets cannot write out of range).
__global__ void atom_struct_kernel(const int* __restrict__ offsets, int S, int N, int* __restrict__ sid) {
  int s = blockIdx.x;
  if (s >= S) return;
  int a0 = max(0, min(N, offsets[s])), a1 = max(0, min(N, offsets[s + 1]));
  for (int a = a0 + threadIdx.x; a < a1; a += blockDim.x) sid[a] = s;
}

// The pinned inclusion test of the pair (i, image (ix, iy, iz) of j): every
// operation rounded to fp32 separately, in the documented order.
__device__ __forceinline__ void image_shift(const float* L, int ix, int iy, int iz, float& sx, float& sy,
                                            float& sz) {
  const float fx = (float)ix, fy = (float)iy, fz = (float)iz;
  sx = __fadd_rn(__fadd_rn(__fmul_rn(fx, L[0]), __fmul_rn(fy, L[3])), __fmul_rn(fz, L[6]));
  sy = __fadd_rn(__fadd_rn(__fmul_rn(fx, L[1]), __fmul_rn(fy, L[4])), __fmul_rn(fz, L[7]));
  sz = __fadd_rn(__fadd_rn(__fmul_rn(fx, L[2]), __fmul_rn(fy, L[5])), __fmul_rn(fz, L[8]));
}
__device__ __forceinline__ bool pair_kept(const float* __restrict__ pos, int i, int j, float xi, float yi, float zi,
                                          float sx, float sy, float sz, bool zero_image, float rc2) {
  const float dx = __fadd_rn(__fsub_rn(pos[3 * j], xi), sx);
  const float dy = __fadd_rn(__fsub_rn(pos[3 * j + 1], yi), sy);
  const float dz = __fadd_rn(__fsub_rn(pos[3 * j + 2], zi), sz);
  const float r2 = __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
  return (r2 < rc2) && !(j == i && zero_image);
}

// Cell list of one structure: the bounding box of its atoms cut into nb[k]
// bins per dimension, each at least r_cut wide, at most n_s bins in all.
struct CellGrid {
  double lo[3];       // lower corner of the box
  double hi[3];       // upper corner
  double inv_w[3];    // bins per unit length (0 for a single bin)
  double margin[3];   // widening of every searched range, far above fp32 rounding
  int nb[3];
  int use;            // 1: the centres of this structure go through the cell-list kernels
};

// Per-centre capacity of the cell-list write pass (sort keys in LDS); a centre
// with more neighbours is written by the all-pairs kernel instead.
constexpr int kCellCap = 512;

// All-pairs search: one wave per centre atom, one neighbour atom j per lane, every image of j
// tested by its lane.  The cell is diagonal (validated before), so the shift of image (ix, iy, iz) is
// (ix Lx, iy Ly, iz Lz) exactly as image_shift rounds it, and r2 = (dx^2 + dy^2) + dz^2 grows
// with each term also when every operation is rounded: an ix (iy) whose dx^2 (dx^2 + dy^2) is not
// below rc^2 has no image to test.  Lanes hold consecutive j and each lists its images in order, so
// an exclusive scan of the lanes' counts gives the canonical order.
// Bound by the vector units.  With candidates (j, image) dealt to lanes and taken apart by 64-bit
// divisions, 256 structures of 8-512 atoms (2.1 M edges, r_cut 6) took 647 us to count and 687 us to
// write; now 44 and 65.
// Centres of structures that use the cell list are skipped (the write pass takes those whose
// neighbours exceed kCellCap).
template <bool WRITE>
__global__ void nl_kernel(const float* __restrict__ pos, const float* __restrict__ cell,
                          const int* __restrict__ offsets, const int* __restrict__ sid, float rc, int N,
                          int* __restrict__ count, const int* __restrict__ rowptr, int* __restrict__ ei,
                          int* __restrict__ ej, int8_t* __restrict__ shift, int* __restrict__ rev,
                          const CellGrid* __restrict__ grid) {
  const int i = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= N) return;
  const int s = sid[i];
  if (grid && grid[s].use && (!WRITE || count[i] <= kCellCap)) return;
  const int a = offsets[s], n = offsets[s + 1] - a;
  const float* L = cell + 9 * s;
  const float Lx = L[0], Ly = L[4], Lz = L[8];
  int mx, my, mz;
  image_range(L, rc, mx, my, mz);
  const float xi = pos[3 * i], yi = pos[3 * i + 1], zi = pos[3 * i + 2];
  const float rc2 = __fmul_rn(rc, rc);
  const int ny = 2 * my + 1, nz = 2 * mz + 1;
  const int packed = ((lane / (ny * nz) - mx) & 255) | ((((lane / nz) % ny - my) & 255) << 8) | ((lane % nz - mz) << 16);
  int base = WRITE ? rowptr[i] : 0;
  int cnt = 0;
  for (int j0 = 0; j0 < n; j0 += 64) {
    const bool live = j0 + lane < n;
    const int j = live ? a + j0 + lane : i;
    const float bx = __fsub_rn(pos[3 * j], xi), by = __fsub_rn(pos[3 * j + 1], yi), bz = __fsub_rn(pos[3 * j + 2], zi);
    // f(image) for every image of j within the cutoff, in order
    auto images = [&](auto f) {
      for (int ix = -mx; ix <= mx; ++ix) {
        const float dx = __fadd_rn(bx, __fmul_rn((float)ix, Lx)), dx2 = __fmul_rn(dx, dx);
        const bool inx = live && dx2 < rc2;
        if (!__any(inx)) continue;
        for (int iy = -my; iy <= my; ++iy) {
          const float dy = __fadd_rn(by, __fmul_rn((float)iy, Ly)), s2 = __fadd_rn(dx2, __fmul_rn(dy, dy));
          const bool iny = inx && s2 < rc2;
          if (!__any(iny)) continue;
          for (int iz = -mz; iz <= mz; ++iz) {
            const float dz = __fadd_rn(bz, __fmul_rn((float)iz, Lz));
            const bool self = j == i && ix == 0 && iy == 0 && iz == 0;
            f(iny && __fadd_rn(s2, __fmul_rn(dz, dz)) < rc2 && !self, ix, iy, iz);
          }
        }
      }
    };
    int c = 0;
    unsigned kept = 0;   // with at most 32 images: bit of every kept one
    images([&](bool keep, int ix, int iy, int iz) {
      c += keep;
      if (WRITE) kept |= (unsigned)keep << ((((ix + mx) * ny + iy + my) * nz + iz + mz) & 31);
    });
    if (!WRITE) {
      cnt += c;
      continue;
    }
    int pre = c;   // inclusive scan over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(pre, o, 64);
      if (lane >= o) pre += v;
    }
    int p = base + pre - c;
    auto put = [&](int ix, int iy, int iz) {
      ei[p] = i;
      ej[p] = j;
      rev[p] = p;
      shift[3LL * p] = (int8_t)ix;
      shift[3LL * p + 1] = (int8_t)iy;
      shift[3LL * p + 2] = (int8_t)iz;
      ++p;
    };
    if ((2 * mx + 1) * ny * nz <= 32) {
      while (__any(kept != 0)) {
        // lane q holds image q, packed
        const int img = __shfl(packed, kept ? __builtin_ctz(kept) : 0, 64);
        if (kept) put((int8_t)img, (int8_t)(img >> 8), (int8_t)(img >> 16));
        kept &= kept - 1;
      }
    } else {
      images([&](bool keep, int ix, int iy, int iz) {
        if (keep) put(ix, iy, iz);
      });
    }
    base += __shfl(pre, 63, 64);
  }
  if (!WRITE) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if (lane == 0) count[i] = cnt;
  }
}

// ------------------------------------------------------------------ cell list
// A structure uses the cell list when mode says so (1: every structure, 2:
// none) or, in mode 0, when its all-pairs candidate count n_s * n_images is at
// least kCellMinCand and its box holds at least 27 bins; without any structure of that
// size the cell-list kernels are not launched.  Bins are built per
// structure from the atoms' own bounding box (positions need not be wrapped);
// a centre then tests, for every image n, only the atoms of the bins that the
// ball of radius r_cut around X_i - s(n) reaches, with the same fp32 test, and
// its kept (j, n) are sorted into the canonical order in LDS: the list is
// bitwise the all-pairs one.

// One workgroup per structure: bounding box, bins, use flag; nbins[s] = bins used.
__global__ void cell_grid_kernel(const float* __restrict__ pos, const float* __restrict__ cell,
                                 const int* __restrict__ offsets, int S, float rc, int mode,
                                 CellGrid* __restrict__ grid, int* __restrict__ nbins) {
  __shared__ float red[6][256];
  const int s = blockIdx.x;
  if (s >= S) return;
  const int a = offsets[s], n = offsets[s + 1] - a;
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int t = threadIdx.x; t < n; t += blockDim.x)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float v = pos[3 * (a + t) + k];
      lo[k] = fminf(lo[k], v);
      hi[k] = fmaxf(hi[k], v);
    }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    red[k][threadIdx.x] = lo[k];
    red[3 + k][threadIdx.x] = hi[k];
  }
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        red[k][threadIdx.x] = fminf(red[k][threadIdx.x], red[k][threadIdx.x + o]);
        red[3 + k][threadIdx.x] = fmaxf(red[3 + k][threadIdx.x], red[3 + k][threadIdx.x + o]);
      }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  CellGrid g;
  const float* L = cell + 9 * s;
  int m[3];
  image_range(L, rc, m[0], m[1], m[2]);
  long long bins = 1;
  for (int k = 0; k < 3; ++k) {
    const double l = n > 0 ? (double)red[k][0] : 0.0, h = n > 0 ? (double)red[3 + k][0] : 0.0;
    const double ext = h - l;
    int nb = (int)fmin(64.0, floor(ext / (double)rc));
    g.nb[k] = nb < 1 ? 1 : nb;
    g.lo[k] = l;
    g.hi[k] = h;
    g.margin[k] = 1e-4 * (fabs(l) + fabs(h) + (m[k] + 1.0) * (double)L[4 * k] + (double)rc);
  }
  // at most n_s bins: halve the widest dimension until the product fits
  while ((long long)g.nb[0] * g.nb[1] * g.nb[2] > (n > 1 ? n : 1)) {
    int k = 0;
    if (g.nb[1] > g.nb[k]) k = 1;
    if (g.nb[2] > g.nb[k]) k = 2;
    g.nb[k] = (g.nb[k] + 1) / 2;
  }
  for (int k = 0; k < 3; ++k) {
    const double ext = n > 0 ? (double)red[3 + k][0] - (double)red[k][0] : 0.0;
    g.inv_w[k] = (g.nb[k] > 1 && ext > 0.0) ? g.nb[k] / ext : 0.0;
  }
  bins = (long long)g.nb[0] * g.nb[1] * g.nb[2];
  const long long nimg = (long long)(2 * m[0] + 1) * (2 * m[1] + 1) * (2 * m[2] + 1);
  int use = 0;
  if (n > 0) use = mode == 1 ? 1 : mode == 2 ? 0 : ((long long)n * nimg >= kCellMinCand && bins >= 27);
  g.use = use;
  grid[s] = g;
  nbins[s] = use ? (int)bins : 0;
}

__device__ __forceinline__ int cell_coord(double x, const CellGrid& g, int k) {
  const double f = floor((x - g.lo[k]) * g.inv_w[k]);
  return f < 0.0 ? 0 : f > g.nb[k] - 1 ? g.nb[k] - 1 : (int)f;
}

// bin of every atom of a cell-list structure, and the atom count of every bin
__global__ void cell_bin_kernel(const float* __restrict__ pos, const int* __restrict__ sid,
                                const CellGrid* __restrict__ grid, const int* __restrict__ bin_off, int N,
                                int* __restrict__ abin, int* __restrict__ bcount) {
  const int at = blockIdx.x * blockDim.x + threadIdx.x;
  if (at >= N) return;
  const int s = sid[at];
  const CellGrid& g = grid[s];
  if (!g.use) return;
  const int bx = cell_coord(pos[3 * at], g, 0), by = cell_coord(pos[3 * at + 1], g, 1),
            bz = cell_coord(pos[3 * at + 2], g, 2);
  const int b = bin_off[s] + (bx * g.nb[1] + by) * g.nb[2] + bz;
  abin[at] = b;
  atomicAdd(bcount + b, 1);
}

// atoms listed by bin (any order inside a bin: the write pass sorts)
__global__ void cell_fill_kernel(const int* __restrict__ sid, const CellGrid* __restrict__ grid,
                                 const int* __restrict__ abin, const int* __restrict__ bstart, int N,
                                 int* __restrict__ bfill, int* __restrict__ batoms) {
  const int at = blockIdx.x * blockDim.x + threadIdx.x;
  if (at >= N) return;
  if (!grid[sid[at]].use) return;
  const int b = abin[at];
  batoms[bstart[b] + atomicAdd(bfill + b, 1)] = at;
}

__device__ __forceinline__ void cell_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per centre of a cell-list structure: count (WRITE = false) or
// collect, sort by (j, image) and write (WRITE = true, at most kCellCap).
template <bool WRITE>
__global__ __launch_bounds__(256) void nl_cell_kernel(
    const float* __restrict__ pos, const float* __restrict__ cell, const int* __restrict__ offsets,
    const int* __restrict__ sid, float rc, int N, const CellGrid* __restrict__ grid, const int* __restrict__ bin_off,
    const int* __restrict__ bstart, const int* __restrict__ batoms, int* __restrict__ count,
    const int* __restrict__ rowptr, int* __restrict__ ei, int* __restrict__ ej, int8_t* __restrict__ shift,
    int* __restrict__ rev) {
  __shared__ unsigned long long keys_all[4][kCellCap];
  const int i = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (i >= N) return;
  const int s = sid[i];
  const CellGrid g = grid[s];
  if (!g.use) return;
  if (WRITE && count[i] > kCellCap) return;
  unsigned long long* keys = keys_all[threadIdx.x >> 6];
  const int a = offsets[s];
  const float* L = cell + 9 * s;
  int mx, my, mz;
  image_range(L, rc, mx, my, mz);
  const int ny = 2 * my + 1, nz = 2 * mz + 1;
  const int nimg = (2 * mx + 1) * ny * nz;
  const float xi = pos[3 * i], yi = pos[3 * i + 1], zi = pos[3 * i + 2];
  const float rc2 = __fmul_rn(rc, rc);
  const int b0 = bin_off[s];
  int cnt = 0;
  for (int im = 0; im < nimg; ++im) {
    const int ix = im / (ny * nz) - mx, iy = (im / nz) % ny - my, iz = im % nz - mz;
    float sx, sy, sz;
    image_shift(L, ix, iy, iz, sx, sy, sz);
    // atoms j near X_i - s(n): bins of the widened ball
    const double c[3] = {(double)xi - (double)sx, (double)yi - (double)sy, (double)zi - (double)sz};
    int lo[3], hi[3];
    bool empty = false;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double r = (double)rc + g.margin[k];
      empty |= c[k] + r < g.lo[k] || c[k] - r > g.hi[k];
      if (g.inv_w[k] == 0.0) {
        lo[k] = hi[k] = 0;
      } else {
        const double f0 = floor((c[k] - r - g.lo[k]) * g.inv_w[k]), f1 = floor((c[k] + r - g.lo[k]) * g.inv_w[k]);
        lo[k] = f0 < 0.0 ? 0 : f0 > g.nb[k] - 1 ? g.nb[k] - 1 : (int)f0;
        hi[k] = f1 < 0.0 ? 0 : f1 > g.nb[k] - 1 ? g.nb[k] - 1 : (int)f1;
      }
    }
    if (empty) continue;
    const bool zero_image = ix == 0 && iy == 0 && iz == 0;
    for (int bx = lo[0]; bx <= hi[0]; ++bx)
      for (int by = lo[1]; by <= hi[1]; ++by)
        for (int bz = lo[2]; bz <= hi[2]; ++bz) {
          const int b = b0 + (bx * g.nb[1] + by) * g.nb[2] + bz;
          const int r0 = bstart[b], r1 = bstart[b + 1];
          for (int t0 = r0; t0 < r1; t0 += 64) {
            const int t = t0 + lane;
            int j = 0;
            bool keep = false;
            if (t < r1) {
              j = batoms[t];
              keep = pair_kept(pos, i, j, xi, yi, zi, sx, sy, sz, zero_image, rc2);
            }
            const unsigned long long m = __ballot(keep);
            if (WRITE && keep) {
              const int p = cnt + __popcll(m & ((1ull << lane) - 1ull));
              if (p < kCellCap) keys[p] = (unsigned long long)(j - a) * (unsigned long long)nimg + (unsigned)im;
            }
            cnt += __popcll(m);
          }
        }
  }
  if (!WRITE) {
    if (lane == 0) count[i] = cnt;
    return;
  }
  cell_wave_sync();
  // rank of every key among the centre's keys (all distinct) = its place in the canonical order
  const int base = rowptr[i];
  for (int q = lane; q < cnt; q += 64) {
    const unsigned long long k = keys[q];
    int r = 0;
    for (int t = 0; t < cnt; ++t) r += keys[t] < k;
    const int p = base + r;
    const int j = a + (int)(k / (unsigned long long)nimg);
    const int im = (int)(k % (unsigned long long)nimg);
    ei[p] = i;
    ej[p] = j;
    rev[p] = p;
    shift[3 * p] = (int8_t)(im / (ny * nz) - mx);
    shift[3 * p + 1] = (int8_t)((im / nz) % ny - my);
    shift[3 * p + 2] = (int8_t)(im % nz - mz);
  }
}

// Exclusive scan of n int32 values into out[0..n]; out[n] is the total and
// totals that do not fit int32 raise flag bit 4.  Three passes over tiles of
// kScanTile values: tile sums, an exclusive scan of the tile sums (one
// workgroup), and the scan of every tile from its offset.  Sums are int64.
constexpr int kScanThreads = 256, kScanPer = 16, kScanTile = kScanThreads * kScanPer;

__device__ __forceinline__ long long block_exclusive_scan(long long v, long long* part, long long& total) {
  const int t = threadIdx.x;
  part[t] = v;
  __syncthreads();
  for (int o = 1; o < kScanThreads; o <<= 1) {
    const long long w = t >= o ? part[t - o] : 0;
    __syncthreads();
    part[t] += w;
    __syncthreads();
  }
  total = part[kScanThreads - 1];
  const long long r = part[t] - v;
  __syncthreads();
  return r;
}

// The same by one workgroup, for inputs of up to kScanOne values, kScanOnePer to a thread: one launch in
// place of three, each of which takes 3 to 5 us whatever its size.  Longer inputs would take a loop, and
// its chain of rounds costs more than it saves (two rounds: whole neighbour list of 32 262 atoms 208.5 us,
// 202.3 by three launches).
constexpr int kScanOneThreads = 1024, kScanOnePer = 16, kScanOne = kScanOneThreads * kScanOnePer;
__global__ __launch_bounds__(kScanOneThreads) void scan_one_kernel(const int* __restrict__ in, int n,
                                                                   int* __restrict__ out, int* __restrict__ flag) {
  __shared__ long long wsum[kScanOneThreads / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int i = kScanOnePer * t;
  int v[kScanOnePer];
  long long s = 0;
  if (i + kScanOnePer <= n) {
#pragma unroll
    for (int k = 0; k < kScanOnePer; k += 4) {
      const int4 u = *reinterpret_cast<const int4*>(in + i + k);
      v[k] = u.x; v[k + 1] = u.y; v[k + 2] = u.z; v[k + 3] = u.w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kScanOnePer; ++k) v[k] = i + k < n ? in[i + k] : 0;
  }
#pragma unroll
  for (int k = 0; k < kScanOnePer; ++k) s += v[k];
  long long inc = s;   // inclusive scan over the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long u = __shfl_up(inc, o, 64);
    if (lane >= o) inc += u;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  long long before = 0, total = 0;
#pragma unroll
  for (int q = 0; q < kScanOneThreads / 64; ++q) {
    if (q < w) before += wsum[q];
    total += wsum[q];
  }
  long long run = before + inc - s;
#pragma unroll
  for (int k = 0; k < kScanOnePer; ++k) {
    if (i + k < n) out[i + k] = (int)run;
    run += v[k];
  }
  if (t == 0) {
    out[n] = (int)total;
    if (total > 0x7fffffffLL && flag) atomicOr(flag, 16);
  }
}

__global__ void scan_tile_sums_kernel(const int* __restrict__ in, int n, long long* __restrict__ sums) {
  __shared__ long long part[kScanThreads];
  const long long lo = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanPer;
  long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k)
    if (lo + k < n) s += in[lo + k];
  long long total;
  block_exclusive_scan(s, part, total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ void scan_sums_kernel(long long* __restrict__ sums, int ntiles, int n, int* __restrict__ out,
                                 int* __restrict__ flag) {
  __shared__ long long part[kScanThreads];
  const int per = (ntiles + kScanThreads - 1) / kScanThreads;
  const int lo = min(ntiles, (int)threadIdx.x * per), hi = min(ntiles, lo + per);
  long long s = 0;
  for (int k = lo; k < hi; ++k) s += sums[k];
  long long total;
  long long run = block_exclusive_scan(s, part, total);
  for (int k = lo; k < hi; ++k) {
    const long long v = sums[k];
    sums[k] = run;
    run += v;
  }
  if (threadIdx.x == 0) {
    out[n] = (int)total;
    if (total > 0x7fffffffLL && flag) atomicOr(flag, 16);
  }
}

__global__ void scan_tile_kernel(const int* __restrict__ in, int n, const long long* __restrict__ offs,
                                 int* __restrict__ out) {
  __shared__ long long part[kScanThreads];
  const long long lo = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanPer;
  int v[kScanPer];
  long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = lo + k < n ? in[lo + k] : 0;
    s += v[k];
  }
  long long total;
  long long run = offs[blockIdx.x] + block_exclusive_scan(s, part, total);
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    if (lo + k < n) out[lo + k] = (int)run;
    run += v[k];
  }
}

// rev[e] = the edge (j, i, -n), found by binary search in the sorted segment of j.  Bound by the
// scattered loads of the search, so only one edge of a pair searches (i < j, or i = j and the first
// non-zero shift positive) and writes both entries: 2.1 M edges 87 us with every edge searching, now 55.
// Every edge has its partner, because the distance test gives the same value both ways (differences and
// shifts only change sign, exactly); the write pass has set rev[e] = e, so that nothing is left unwritten.
__global__ void reverse_kernel(const int* __restrict__ ei, const int* __restrict__ ej,
                               const int8_t* __restrict__ shift, const int* __restrict__ rowptr, int Ne,
                               int* __restrict__ rev) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Ne) return;
  const int i = ei[e], j = ej[e];
  if (i > j) return;
  const int kx = -shift[3LL * e], ky = -shift[3LL * e + 1], kz = -shift[3LL * e + 2];
  if (i == j && (kx != 0 ? kx > 0 : ky != 0 ? ky > 0 : kz > 0)) return;
  // key of an edge within the segment of j: (ej, sx, sy, sz) lexicographic
  auto less = [&](int f) {
    int fj = ej[f];
    if (fj != i) return fj < i;
    int fx = shift[3LL * f], fy = shift[3LL * f + 1], fz = shift[3LL * f + 2];
    if (fx != kx) return fx < kx;
    if (fy != ky) return fy < ky;
    return fz < kz;
  };
  int lo = rowptr[j], hi = rowptr[j + 1];
  const int end = hi;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (less(mid)) lo = mid + 1; else hi = mid;
  }
  const bool ok = lo < end && ej[lo] == i && shift[3LL * lo] == kx && shift[3LL * lo + 1] == ky &&
                  shift[3LL * lo + 2] == kz;
  if (ok) {
    rev[e] = lo;
    rev[lo] = e;
  }
}

// Edge geometry in float64 from the fp32 inputs, then stored as fp32:
// d = X_j + n.L - X_i, r = |d|, u = d / r, and the Bessel basis with the p = 6
// polynomial envelope and its radial derivative,
//   B_n(r)  = sqrt(2/rc) sin(n pi r / rc) / r * u(r / rc),
//   u(x)    = 1 - 28 x^6 + 48 x^7 - 21 x^8   (x < 1).
// Envelope u(r / rc) and its radial derivative (zero beyond the cutoff).
__device__ __forceinline__ void envelope_at(double r, double rcd, double& u, double& du) {
  const double x = r / rcd;
  u = 0.0;
  du = 0.0;
  if (x < 1.0) {
    const double x2 = x * x, x5 = x2 * x2 * x, x6 = x5 * x;
    u = 1.0 - 28.0 * x6 + 48.0 * x6 * x - 21.0 * x6 * x2;
    du = (-168.0 * x5 + 336.0 * x6 - 168.0 * x6 * x) / rcd;
  }
}

// B_n(r) and dB_n/dr, n = 1..nb, for cutoff rc, into B[0..nb), dB[0..nb).
__device__ __forceinline__ void bessel_at(double r, double rcd, int nb, float* __restrict__ B,
                                          float* __restrict__ dB) {
  double u, du;
  envelope_at(r, rcd, u, du);
  const double c = sqrt(2.0 / rcd);
  const double th = M_PI / rcd;
  // sin(n x), cos(n x) for x = th r by the angle-addition identities from one sincos
  // (float64: the recurrence's rounding stays far below the float32 outputs')
  double s1, c1;
  sincos(th * r, &s1, &c1);
  double sn = s1, cs = c1;
  const double ir = 1.0 / r;
  // nb is a multiple of 4 and the rows 16-byte aligned: four values per store
  for (int n0 = 1; n0 <= nb; n0 += 4) {
    float b[4], db[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double k = (n0 + q) * th;
      const double s = sn * ir;
      const double ds = (k * cs - s) * ir;
      b[q] = (float)(c * s * u);
      db[q] = (float)(c * (ds * u + s * du));
      const double sn1 = sn * c1 + cs * s1;
      cs = cs * c1 - sn * s1;
      sn = sn1;
    }
    *reinterpret_cast<float4*>(B + n0 - 1) = make_float4(b[0], b[1], b[2], b[3]);
    *reinterpret_cast<float4*>(dB + n0 - 1) = make_float4(db[0], db[1], db[2], db[3]);
  }
}

// d2B_n/dr2, n = 1..nb, for cutoff rc (the loss gradient in positions needs the
// second radial derivative of the basis):
//   B = c s u,  s = sin(k r) / r,  s' = (k cos(k r) - s) / r,  s'' = -k^2 s - 2 s' / r,
//   B'' = c (s'' u + 2 s' u' + s u''),  u'' = (-840 x^4 + 2016 x^5 - 1176 x^6) / rc^2.
__device__ __forceinline__ void bessel_d2_at(double r, double rcd, int nb, float* __restrict__ d2B) {
  double u, du;
  envelope_at(r, rcd, u, du);
  const double x = r / rcd;
  double d2u = 0.0;
  if (x < 1.0) {
    const double x2 = x * x, x4 = x2 * x2;
    d2u = (-840.0 * x4 + 2016.0 * x4 * x - 1176.0 * x4 * x2) / (rcd * rcd);
  }
  const double c = sqrt(2.0 / rcd);
  const double th = M_PI / rcd;
  double s1, c1;
  sincos(th * r, &s1, &c1);
  double sn = s1, cs = c1;
  const double ir = 1.0 / r;
  for (int n0 = 1; n0 <= nb; n0 += 4) {
    float b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double k = (n0 + q) * th;
      const double s = sn * ir;
      const double ds = (k * cs - s) * ir;
      const double d2s = -k * k * s - 2.0 * ds * ir;
      b[q] = (float)(c * (d2s * u + 2.0 * ds * du + s * d2u));
      const double sn1 = sn * c1 + cs * s1;
      cs = cs * c1 - sn * s1;
      sn = sn1;
    }
    *reinterpret_cast<float4*>(d2B + n0 - 1) = make_float4(b[0], b[1], b[2], b[3]);
  }
}

// With rc3 > 0 also the three-body basis B3, dB3 (cutoff rc3) and the
// envelope u(r / rc3) with its derivative, per edge; with d2B also B''.
__global__ void geometry_kernel(const float* __restrict__ pos, const float* __restrict__ cell,
                                const int* __restrict__ sid, const int* __restrict__ ei,
                                const int* __restrict__ ej, const int8_t* __restrict__ shift, int Ne,
                                float rc, int nb, float4* __restrict__ geo, float* __restrict__ B,
                                float* __restrict__ dB, float rc3, float* __restrict__ B3, float* __restrict__ dB3,
                                float* __restrict__ u3, float* __restrict__ du3, float* __restrict__ d2B) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Ne) return;
  const int i = ei[e], j = ej[e];
  const float* L = cell + 9 * sid[i];
  const double nx = shift[3 * e], ny = shift[3 * e + 1], nz = shift[3 * e + 2];
  double d[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    d[k] = ((double)pos[3 * j + k] - (double)pos[3 * i + k]) +
           (nx * (double)L[k] + ny * (double)L[3 + k] + nz * (double)L[6 + k]);
  const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  geo[e] = make_float4((float)(d[0] / r), (float)(d[1] / r), (float)(d[2] / r), (float)r);
  bessel_at(r, (double)rc, nb, B + (long long)e * nb, dB + (long long)e * nb);
  if (d2B) bessel_d2_at(r, (double)rc, nb, d2B + (long long)e * nb);
  if (rc3 > 0.f) {
    bessel_at(r, (double)rc3, nb, B3 + (long long)e * nb, dB3 + (long long)e * nb);
    double u, du;
    envelope_at(r, (double)rc3, u, du);
    u3[e] = (float)u;
    du3[e] = (float)du;
  }
}

void launch_validate_struct(hipStream_t st, const int* offsets, int S, int N, const float* cell, float rc,
                            int* flag) {
  hipLaunchKernelGGL(validate_struct_kernel, dim3(cdiv(S + 1, 256)), dim3(256), 0, st, offsets, S, N, cell,
                     rc, flag);
}

void launch_atom_struct(hipStream_t st, const int* offsets, int S, int N, int* sid) {
  hipLaunchKernelGGL(atom_struct_kernel, dim3(S), dim3(256), 0, st, offsets, S, N, sid);
}

// scratch: cdiv(n, kScanTile) int64 values (scan_scratch_bytes)
size_t scan_scratch_bytes(long long n) { return sizeof(long long) * (size_t)((n + kScanTile - 1) / kScanTile + 1); }

void launch_exclusive_scan(hipStream_t st, const int* in, int n, int* out, int* flag, long long* scratch) {
  if (n <= kScanOne) {
    hipLaunchKernelGGL(scan_one_kernel, dim3(1), dim3(kScanOneThreads), 0, st, in, n, out, flag);
    return;
  }
  const int ntiles = (int)cdiv(n, kScanTile);
  if (ntiles > 0) {
    hipLaunchKernelGGL(scan_tile_sums_kernel, dim3(ntiles), dim3(kScanThreads), 0, st, in, n, scratch);
  }
  hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kScanThreads), 0, st, scratch, ntiles, n, out, flag);
  if (ntiles > 0) {
    hipLaunchKernelGGL(scan_tile_kernel, dim3(ntiles), dim3(kScanThreads), 0, st, in, n, (const long long*)scratch,
                       out);
  }
}

void launch_geometry(hipStream_t st, const float* pos, const float* cell, const int* sid, const int* ei,
                     const int* ej, const int8_t* shift, int Ne, float rc, int nb, float4* geo, float* B,
                     float* dB, float rc3, float* B3, float* dB3, float* u3, float* du3, float* d2B) {
  if (Ne <= 0) return;
  hipLaunchKernelGGL(geometry_kernel, dim3(cdiv(Ne, 256)), dim3(256), 0, st, pos, cell, sid, ei, ej, shift, Ne,
                     rc, nb, geo, B, dB, rc3, B3, dB3, u3, du3, d2B);
}

}  // namespace janus

using namespace janus;

extern "C" int janus_set_edge_builder(janus_ctx* ctx, int32_t mode) {
  if (!ctx || mode < 0 || mode > 2) return JANUS_EINVAL;
  ctx->edge_builder = mode;
  return JANUS_OK;
}

extern "C" int janus_build_edges(janus_ctx* ctx, const float* pos, const float* cell, const int32_t* offsets,
                                 int32_t n_atoms, int32_t n_struct, int64_t capacity, int32_t* ei, int32_t* ej,
                                 int8_t* shift, int32_t* rowptr, int32_t* rev, int64_t* n_edges, void* stream) {
  if (!ctx || !pos || !cell || !offsets || !rowptr || !n_edges || n_atoms < 1 || n_struct < 1 || capacity < 0)
    return JANUS_EINVAL;
  if (capacity > 0 && (!ei || !ej || !shift || !rev)) return JANUS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int N = n_atoms, S = n_struct;
  const long long scan_n = N > S ? N : S;
  auto carve = [&](Carver& c, int*& flag, int*& sid, int*& count, int*& rp, long long*& scan, CellGrid*& grid,
                   int*& nbins, int*& bin_off, int*& abin, int*& bcount, int*& bstart, int*& bfill, int*& batoms) {
    flag = c.take<int>(1);
    sid = c.take<int>(N);
    count = c.take<int>(N);
    rp = c.take<int>(N + 1);
    scan = c.take<long long>(scan_scratch_bytes(scan_n) / sizeof(long long));
    grid = c.take<CellGrid>(S);
    nbins = c.take<int>(S);
    bin_off = c.take<int>(S + 1);
    abin = c.take<int>(N);
    bcount = c.take<int>(N);
    bstart = c.take<int>(N + 1);
    bfill = c.take<int>(N);
    batoms = c.take<int>(N);
  };
  int *flag, *sid, *count, *rp, *nbins, *bin_off, *abin, *bcount, *bstart, *bfill, *batoms;
  long long* scan;
  CellGrid* grid;
  Carver cv(nullptr);
  carve(cv, flag, sid, count, rp, scan, grid, nbins, bin_off, abin, bcount, bstart, bfill, batoms);
  int rc = ensure(ctx->nl, cv.size());
  if (rc) return rc;
  Carver c2(ctx->nl.ptr);
  carve(c2, flag, sid, count, rp, scan, grid, nbins, bin_off, abin, bcount, bstart, bfill, batoms);
  int* hw = ctx->host_word;

  JANUS_HIP_TRY(hipMemsetAsync(flag, 0, sizeof(int), st));
  launch_validate_struct(st, offsets, S, N, cell, ctx->cfg.r_cut, flag);
  launch_atom_struct(st, offsets, S, N, sid);
  JANUS_HIP_TRY(hipGetLastError());
  JANUS_HIP_TRY(hipMemcpyAsync(hw, flag, sizeof(int), hipMemcpyDeviceToHost, st));
  JANUS_HIP_TRY(hipStreamSynchronize(st));
  if (hw[0] & 1) return JANUS_EINVAL;
  if (hw[0] & 2) return JANUS_EUNSUPPORTED;
  const bool cells = ctx->edge_builder == 1 || (ctx->edge_builder == 0 && (hw[0] & 32));

  const float r_cut = ctx->cfg.r_cut;
  const dim3 gw(cdiv((long long)N * 64, 256)), b256(256);
  {
    ProfScope ps(ctx, st, PROF_GRAPH, 0.0, 16.0 * N);
    // cell lists of the structures that use them (none in mode 2, or without a large structure in mode 0)
    if (!cells) grid = nullptr;
    if (cells) {
      hipLaunchKernelGGL(cell_grid_kernel, dim3(S), b256, 0, st, pos, cell, offsets, S, r_cut, ctx->edge_builder, grid,
                         nbins);
      launch_exclusive_scan(st, nbins, S, bin_off, flag, scan);
      JANUS_HIP_TRY(hipMemsetAsync(bcount, 0, sizeof(int) * N, st));
      JANUS_HIP_TRY(hipMemsetAsync(bfill, 0, sizeof(int) * N, st));
      hipLaunchKernelGGL(cell_bin_kernel, dim3(cdiv(N, 256)), b256, 0, st, pos, sid, grid, bin_off, N, abin, bcount);
      launch_exclusive_scan(st, bcount, N, bstart, flag, scan);
      hipLaunchKernelGGL(cell_fill_kernel, dim3(cdiv(N, 256)), b256, 0, st, sid, grid, abin, bstart, N, bfill,
                         batoms);
      hipLaunchKernelGGL((nl_cell_kernel<false>), gw, b256, 0, st, pos, cell, offsets, sid, r_cut, N, grid, bin_off,
                         bstart, batoms, count, nullptr, nullptr, nullptr, nullptr, nullptr);
    }
    hipLaunchKernelGGL((nl_kernel<false>), gw, b256, 0, st, pos, cell, offsets, sid, r_cut, N, count, nullptr,
                       nullptr, nullptr, nullptr, nullptr, grid);
    launch_exclusive_scan(st, count, N, rp, flag, scan);
  }
  JANUS_HIP_TRY(hipGetLastError());
  JANUS_HIP_TRY(hipMemcpyAsync(hw, rp + N, sizeof(int), hipMemcpyDeviceToHost, st));
  JANUS_HIP_TRY(hipMemcpyAsync(hw + 1, flag, sizeof(int), hipMemcpyDeviceToHost, st));
  JANUS_HIP_TRY(hipStreamSynchronize(st));
  if (hw[1] & 16) return JANUS_EUNSUPPORTED;   // more than 2^31 - 1 edges
  const long long ne = hw[0];
  *n_edges = ne;
  if (ne > capacity) return JANUS_ECAPACITY;
  JANUS_HIP_TRY(hipMemcpyAsync(rowptr, rp, sizeof(int) * (N + 1), hipMemcpyDeviceToDevice, st));
  if (ne > 0) {
    ProfScope ps(ctx, st, PROF_GRAPH, 0.0, 16.0 * N + 23.0 * ne);
    if (cells)
      hipLaunchKernelGGL((nl_cell_kernel<true>), gw, b256, 0, st, pos, cell, offsets, sid, r_cut, N, grid, bin_off,
                         bstart, batoms, count, rp, ei, ej, shift, rev);
    hipLaunchKernelGGL((nl_kernel<true>), gw, b256, 0, st, pos, cell, offsets, sid, r_cut, N, count, rp, ei, ej,
                       shift, rev, grid);
    hipLaunchKernelGGL(reverse_kernel, dim3(cdiv(ne, 256)), dim3(256), 0, st, ei, ej, shift, rp, (int)ne, rev);
  }
  JANUS_HIP_TRY(hipGetLastError());
  return JANUS_OK;
}
