// tile_kernels.hip -- sums, copies and updates between per-tile buffers: the
// neighbour addition and the directional passes of Sections III and IV, the
// stitches, and the tile updates of Alg. 1.  All are bound by memory traffic,
// so each kernel takes a whole list of boxes: one launch per stage instead of
// one per pair of boxes, and every destination value is written once with its
// sources summed in registers in the given order.
#include "ptycho_kernels.h"

namespace ptycho {

namespace {

constexpr int kWaves = 4;  // waves per workgroup; a wave walks rows, its lanes columns
constexpr int kCols = 4;   // columns per lane and step of the updates, loaded together
// The same of the box lists.  2 / 4 / 8 / 10 took 589 / 580 / 577 / 570 us for neighbour addition and stitch of
// 16 boxes 640 wide (16 slices), 206 / 192 / 180 / 181 for 320 to 384 wide, 481 / 471 / 465 / 463 for 4 boxes 1088
// wide, 204 / 195 / 188 / 189 for 950 wide (8 slices); for narrower or fewer values they are alike.
constexpr int kBoxCols = 10;

// One box operation per (blockIdx.y / S), one slice of it per blockIdx.y % S.
// Bound: the bytes of the boxes.  The neighbour addition of 16 boxes of 640^2 x
// 16 slices and the stitch of their interiors took 116 launches and 1.08 ms on
// the device (each too small to fill it; 1.46 ms with the gaps), as lists 3
// launches and 0.57 ms (3.6 TB/s); the sum of the 16 boxes into the gradient
// 0.56 ms as a fill and 16 additions, 0.27 ms as a list.
__global__ void __launch_bounds__(64 * kWaves) box_list_kernel(BoxList list, int S) {
  const int o = static_cast<int>(blockIdx.y) / S, s = static_cast<int>(blockIdx.y) % S;
  const BoxOp op = list.op[o];
  const int lane = static_cast<int>(threadIdx.x & 63);
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  for (int y = static_cast<int>(blockIdx.x) * kWaves + wave; y < op.h; y += static_cast<int>(gridDim.x) * kWaves) {
    float2* __restrict__ drow = op.dst + s * op.slice + static_cast<long long>(y) * op.ld;
    for (int xb = lane; xb < op.w; xb += 64 * kBoxCols) {
      float2 a[kBoxCols];
      if (op.init == kBoxAdd) {
        for (int k = 0; k < kBoxCols; ++k) a[k] = xb + 64 * k < op.w ? drow[xb + 64 * k] : make_float2(0.f, 0.f);
      } else {
        for (int k = 0; k < kBoxCols; ++k) a[k] = make_float2(0.f, 0.f);
      }
      for (int i = 0; i < op.nsrc; ++i) {
        const BoxSrc& src = list.src[op.first + i];
        if (y < src.y0 || y >= src.y1) continue;  // uniform
        const float2* __restrict__ srow = src.p + s * src.slice + static_cast<long long>(y) * src.ld;
        float2 v[kBoxCols];
        bool in[kBoxCols];
        for (int k = 0; k < kBoxCols; ++k) {
          const int x = xb + 64 * k;
          in[k] = x >= src.x0 && x < src.x1;
          v[k] = in[k] ? srow[x] : make_float2(0.f, 0.f);
        }
        if (op.init == kBoxCopy && i == 0) {
          for (int k = 0; k < kBoxCols; ++k) a[k] = v[k];
        } else {
          for (int k = 0; k < kBoxCols; ++k)
            if (in[k]) a[k] = make_float2(a[k].x + v[k].x, a[k].y + v[k].y);
        }
      }
      for (int k = 0; k < kBoxCols; ++k)
        if (xb + 64 * k < op.w) drow[xb + 64 * k] = a[k];
    }
  }
}

// Part of a tile table from the kernel arguments to device memory, word by word.
__global__ void __launch_bounds__(256) set_tiles_kernel(TileChunk chunk, int ntiles, TileDesc* __restrict__ dst) {
  constexpr int kWords = sizeof(TileDesc) / sizeof(int);
  const int* src = reinterpret_cast<const int*>(chunk.t);
  int* out = reinterpret_cast<int*>(dst);
  for (int i = static_cast<int>(threadIdx.x); i < ntiles * kWords; i += 256) out[i] = src[i];
}

__device__ __forceinline__ int wave_min(int v) {
  for (int o = 32; o > 0; o >>= 1) {
    const int u = __shfl_xor(v, o);
    v = u < v ? u : v;
  }
  return v;
}

// One batch of Alg. 1 for every tile of a chunk (blockIdx.y, blockIdx.z = slice): AccBuf += g,
// V -= step * g and g = 0, on the bounding box of the windows that the tile's
// batch touched; g is zero elsewhere, so the rest would not change.  Bound: six
// accesses per value of that box; the whole extended boxes in separate passes
// (zero, two axpy) moved 4 to 5 times as much for 64 positions per tile (31 us
// per batch of 4 tiles of 576^2 x 8 slices instead of 150).  The
// first workgroup of a tile also sums its losses, in a fixed order.  The lists are device data: an entry
// that the gradient launch skips (no such position, listed under another tile than its own, outside the
// box) takes no part here, and a segment is cut to the batch.
__global__ void __launch_bounds__(64 * kWaves) tile_step_kernel(TileChunk tiles, int tile0, int M,
                                                               const int* __restrict__ pos,
                                                               const int* __restrict__ tile_of_pos, int total,
                                                               const int* __restrict__ index, int n,
                                                               const int* __restrict__ seg, float step,
                                                               const double* __restrict__ loss_work,
                                                               double* __restrict__ losses) {
  __shared__ int box[4][kWaves];
  __shared__ double part[64 * kWaves];
  const int k = tile0 + static_cast<int>(blockIdx.y), s = static_cast<int>(blockIdx.z);
  const TileDesc T = tiles.t[blockIdx.y];
  const int lo = max(seg[k], 0), hi = min(seg[k + 1], n);
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (blockIdx.x == 0 && s == 0) {  // uniform
    double f = 0.0;
    for (int i = lo + tid; i < hi; i += 64 * kWaves) f += loss_work[i];
    part[tid] = f;
    __syncthreads();
    for (int w = 32 * kWaves; w > 0; w >>= 1) {
      if (tid < w) part[tid] += part[tid + w];
      __syncthreads();
    }
    if (tid == 0) losses[k] = part[0];
  }
  if (lo >= hi) return;
  int y0 = T.eh, x0 = T.ew, ny1 = 0, nx1 = 0;  // box-local corner minima, and minus the maxima
  for (int i = lo + tid; i < hi; i += 64 * kWaves) {
    const int p = index[i];
    if (p < 0 || p >= total || tile_of_pos[p] != k) continue;  // skipped by the gradient launch too, as the next
    const int gy = pos[2 * p], gx = pos[2 * p + 1];
    if (gy < T.ey0 || gx < T.ex0 || gy > T.ey0 + T.eh - M || gx > T.ex0 + T.ew - M) continue;
    const int y = gy - T.ey0, x = gx - T.ex0;
    y0 = y < y0 ? y : y0;
    x0 = x < x0 ? x : x0;
    ny1 = -(y + M) < ny1 ? -(y + M) : ny1;
    nx1 = -(x + M) < nx1 ? -(x + M) : nx1;
  }
  y0 = wave_min(y0);
  x0 = wave_min(x0);
  ny1 = wave_min(ny1);
  nx1 = wave_min(nx1);
  if (lane == 0) {
    box[0][wave] = y0;
    box[1][wave] = x0;
    box[2][wave] = ny1;
    box[3][wave] = nx1;
  }
  __syncthreads();
  for (int w = 0; w < kWaves; ++w) {
    y0 = box[0][w] < y0 ? box[0][w] : y0;
    x0 = box[1][w] < x0 ? box[1][w] : x0;
    ny1 = box[2][w] < ny1 ? box[2][w] : ny1;
    nx1 = box[3][w] < nx1 ? box[3][w] : nx1;
  }
  for (int y = y0 + static_cast<int>(blockIdx.x) * kWaves + wave; y < -ny1; y += static_cast<int>(gridDim.x) * kWaves) {
    const long long row = s * T.gslice + static_cast<long long>(y) * T.gld;
    float2* __restrict__ g = T.grad + row;
    float2* __restrict__ v = T.obj + row;
    float2* __restrict__ a = T.acc + row;
    for (int xb = x0 + lane; xb < -nx1; xb += 64 * kCols) {
      float2 dg[kCols], dv[kCols], da[kCols];
      for (int c = 0; c < kCols; ++c) {
        const int x = xb + 64 * c;
        if (x < -nx1) {
          dg[c] = g[x];
          dv[c] = v[x];
          da[c] = a[x];
        }
      }
      for (int c = 0; c < kCols; ++c) {
        const int x = xb + 64 * c;
        if (x < -nx1) {
          a[x] = make_float2(da[c].x + dg[c].x, da[c].y + dg[c].y);
          v[x] = make_float2(dv[c].x - step * dg[c].x, dv[c].y - step * dg[c].y);
          g[x] = make_float2(0.f, 0.f);
        }
      }
    }
  }
}

// The accumulated update of Alg. 1 for every tile of a chunk (blockIdx.y, blockIdx.z = slice):
// V -= step * AccBuf, AccBuf = 0.  Bound: four accesses per value.
__global__ void __launch_bounds__(64 * kWaves) tile_flush_kernel(TileChunk tiles, float step) {
  const int s = static_cast<int>(blockIdx.z);
  const TileDesc T = tiles.t[blockIdx.y];
  const long long n = static_cast<long long>(T.eh) * T.ew;  // dense
  float2* __restrict__ v = T.obj + s * T.gslice;
  float2* __restrict__ a = T.acc + s * T.gslice;
  for (long long i = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<long long>(gridDim.x) * blockDim.x) {
    const float2 da = a[i], dv = v[i];
    v[i] = make_float2(dv.x - step * da.x, dv.y - step * da.y);
    a[i] = make_float2(0.f, 0.f);
  }
}

}  // namespace

hipError_t launch_box_list(const BoxList& list, int S, int rows, hipStream_t st) {
  if (list.nops == 0) return hipSuccess;
  // two rows per wave: enough workgroups for one box, few enough scalar set-ups for many
  const unsigned gx = static_cast<unsigned>((rows + 2 * kWaves - 1) / (2 * kWaves));
  hipLaunchKernelGGL(box_list_kernel, dim3(gx, static_cast<unsigned>(list.nops * S)), dim3(64 * kWaves), 0, st, list, S);
  return hipGetLastError();
}

namespace {
// Launches over the tiles, as many at a time as a chunk holds: f(chunk, first tile, tiles).
template <class F>
hipError_t for_chunks(const TileDesc* tiles, int ntiles, F&& f) {
  for (int k = 0; k < ntiles; k += TileChunk::kTiles) {
    const int n = ntiles - k < TileChunk::kTiles ? ntiles - k : TileChunk::kTiles;
    TileChunk c;
    for (int i = 0; i < n; ++i) c.t[i] = tiles[k + i];
    f(c, k, n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
}  // namespace

hipError_t launch_set_tiles(const TileDesc* tiles, int ntiles, TileDesc* dev, hipStream_t st) {
  return for_chunks(tiles, ntiles, [&](const TileChunk& c, int k, int n) {
    hipLaunchKernelGGL(set_tiles_kernel, dim3(1), dim3(256), 0, st, c, n, dev + k);
  });
}

hipError_t launch_tile_step(const TileDesc* tiles, int ntiles, int S, int M, const int* pos, const int* tile_of_pos,
                            int total, const int* index, int n, const int* seg, float step, const double* loss_work,
                            double* losses, hipStream_t st) {
  return for_chunks(tiles, ntiles, [&](const TileChunk& c, int k, int m) {
    hipLaunchKernelGGL(tile_step_kernel, dim3(32, static_cast<unsigned>(m), static_cast<unsigned>(S)),
                       dim3(64 * kWaves), 0, st, c, k, M, pos, tile_of_pos, total, index, n, seg, step, loss_work,
                       losses);
  });
}

hipError_t launch_tile_flush(const TileDesc* tiles, int ntiles, int S, float step, hipStream_t st) {
  return for_chunks(tiles, ntiles, [&](const TileChunk& c, int, int m) {
    hipLaunchKernelGGL(tile_flush_kernel, dim3(64, static_cast<unsigned>(m), static_cast<unsigned>(S)),
                       dim3(64 * kWaves), 0, st, c, step);
  });
}

}  // namespace ptycho
