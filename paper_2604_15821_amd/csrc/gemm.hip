// Tables, chunk reduction and the standalone grouped-GEMM entry points.
#include <cstring>
#include <mutex>

#include "internal.h"

namespace janus {

// Tables of one or several grouped products: workgroup x builds job x's, for block y of the job's
// strides.  Group sizes come from the row offsets, from token totals (the offsets are then
// written too) or, with neither, from one group of `rows` rows.  Every launch of this kernel takes 2 to
// 3 us whatever it builds, so all tables that are ready together share one.
__global__ __launch_bounds__(256) void build_tables_kernel(TableJobs jobs) {
  __shared__ int off[1025], tpre[1025], cpre[1025];
  const TableJob j = jobs.job[blockIdx.x];
  const long long y = blockIdx.y;
  const int n = j.groups;
  if (j.totals) {
    if ((int)threadIdx.x < n) tpre[threadIdx.x] = j.totals[y * n + threadIdx.x];   // at most 64 experts
    __syncthreads();
    if (threadIdx.x == 0) {
      int acc = 0;
      for (int g = 0; g < n; ++g) {
        off[g] = acc;
        acc += tpre[g];
      }
      off[n] = acc;
    }
    __syncthreads();
    if ((int)threadIdx.x <= n) j.off_out[y * (n + 1) + threadIdx.x] = off[threadIdx.x];
  } else {
    for (int g = threadIdx.x; g <= n; g += blockDim.x) off[g] = j.off ? j.off[y * (n + 1) + g] : g ? j.rows : 0;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    int t = 0, c = 0;
    for (int g = 0; g < n; ++g) {
      const int m = off[g + 1] - off[g];
      tpre[g] = t;
      cpre[g] = c;
      t += (m + GBM - 1) / GBM;
      if (j.chunks) c += (m + j.kc - 1) / j.kc;
    }
    tpre[n] = t;
    cpre[n] = c;
  }
  __syncthreads();
  auto find = [&](const int* pre, int q) {   // the group g with pre[g] <= q < pre[g + 1]
    int lo = 0, hi = n;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid] <= q) lo = mid; else hi = mid;
    }
    return lo;
  };
  if (j.tiles) {
    if (threadIdx.x == 0) j.n_tiles[y] = tpre[n];
    for (int q = threadIdx.x; q < tpre[n]; q += blockDim.x) {
      const int g = find(tpre, q);
      j.tiles[y * j.tile_stride + q] = RowsTile{g, off[g] + (q - tpre[g]) * GBM, off[g + 1], 0};
    }
  }
  if (j.chunks) {
    if (threadIdx.x == 0) j.n_chunks[y] = cpre[n];
    for (int g = threadIdx.x; g <= n; g += blockDim.x) j.chunk_first[y * (n + 1) + g] = cpre[g];
    for (int q = threadIdx.x; q < cpre[n]; q += blockDim.x) {
      const int g = find(cpre, q), r0 = off[g] + (q - cpre[g]) * j.kc;
      j.chunks[y * j.chunk_stride + q] = WChunk{g, r0, min(r0 + j.kc, off[g + 1]), cpre[g + 1] - cpre[g] == 1};
    }
  }
}

// G_g (+)= sum of the chunk partials of group g.  A workgroup owns 16
// float4 columns; its 16 column-slices sum the chunks c0 + s, c0 + s + 16, ...
// (two accumulators each), and the slices are added in order 0..15, so the
// result is the same on every run.
constexpr int kRedSlices = 16;
__global__ void wgrad_reduce_kernel(const float* __restrict__ partial, const int* __restrict__ chunk_first,
                                    int n_groups, long long PQ, float* __restrict__ G, int accumulate,
                                    bool alone_done) {
  __shared__ float4 red[kRedSlices][16];
  const int g = blockIdx.y;
  const int cl = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const long long i4 = (long long)blockIdx.x * 16 + cl;
  const bool ok = 4 * i4 < PQ;
  const int c0 = chunk_first[g], c1 = chunk_first[g + 1];
  if (alone_done && (c1 - c0 == 1 || (c1 == c0 && accumulate))) return;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
  if (ok) {
    int c = c0 + sl;
    for (; c + kRedSlices < c1; c += 2 * kRedSlices) {
      const float4 u = reinterpret_cast<const float4*>(partial + (long long)c * PQ)[i4];
      const float4 v = reinterpret_cast<const float4*>(partial + (long long)(c + kRedSlices) * PQ)[i4];
      a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
      b.x += v.x; b.y += v.y; b.z += v.z; b.w += v.w;
    }
    if (c < c1) {
      const float4 u = reinterpret_cast<const float4*>(partial + (long long)c * PQ)[i4];
      a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
    }
  }
  red[sl][cl] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
  __syncthreads();
  if (sl == 0 && ok) {
    float4* out = reinterpret_cast<float4*>(G + (long long)g * PQ) + i4;
    float4 s = accumulate ? *out : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < kRedSlices; ++q) {
      const float4 v = red[q][cl];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    *out = s;
  }
}

int skinny_chunk_rows(long long M, int P, int Q) {
  const size_t lds = sizeof(float) * P * Q;
  int per_cu = 0, dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, skinny_kernel(P, Q), 256, lds);
  const long long slots = (e == hipSuccess && per_cu > 0 && cus > 0) ? (long long)per_cu * cus : 1024;
  const long long R = skinny_rows(Q);
  const long long per = (M + slots - 1) / slots;
  const long long kc = ((per + R - 1) / R) * R;
  return (int)(kc < R ? R : kc);
}

void launch_wgrad_reduce(hipStream_t st, const float* partial, const int* chunk_first, int groups,
                         long long PQ, float* G, int accumulate, bool alone_done) {
  dim3 rg(cdiv(PQ / 4, 16), groups);
  hipLaunchKernelGGL(wgrad_reduce_kernel, rg, dim3(16 * kRedSlices), 0, st, partial, chunk_first, groups, PQ, G,
                     accumulate, alone_done);
}

void build_tables(hipStream_t st, const TableJobs& jobs, int n_jobs, int n_blocks) {
  hipLaunchKernelGGL(build_tables_kernel, dim3(n_jobs, n_blocks), dim3(256), 0, st, jobs);
}

// The standalone product.  Up to 64 groups and four rounds of resident workgroups, each works its
// tile out of the offsets (no table launch, about 4 us); a longer grid reads it from a table.
static void grouped_rows(hipStream_t st, const float* A, const float* B, float* C, const int32_t* row_off,
                         int n_groups, int K, int N, int trans_b, RowsTile* tiles, int* nt, int mt) {
  RowsTable table{tiles, nt, row_off, n_groups};
  if (n_groups <= 64 && (long long)mt * ((N + GBN - 1) / GBN) <= 2048)
    table.tiles = nullptr;
  else
    build_tables(st, tables_of(row_off, n_groups).rows_tiles(tiles, nt));
  if (trans_b)
    launch_rows<true>(std::true_type{}, st, LoadPlain{A, K}, B, K, N, table, mt, EpiStore{C, N});
  else
    launch_rows<false>(std::true_type{}, st, LoadPlain{A, K}, B, K, N, table, mt, EpiStore{C, N});
}

int ensure(janus_buffer& b, size_t bytes) {
  if (bytes <= b.bytes && b.ptr) return JANUS_OK;
  if (b.ptr) {
    hipError_t e = hipFree(b.ptr);
    b.ptr = nullptr;
    b.bytes = 0;
    if (e != hipSuccess) return janus_set_hip_error(e);
  }
  size_t want = bytes < 256 ? 256 : bytes;
  if (hipMalloc(&b.ptr, want) != hipSuccess) {
    (void)hipGetLastError();
    b.ptr = nullptr;
    return JANUS_ENOMEM;
  }
  b.bytes = want;
  return JANUS_OK;
}

}  // namespace janus

using namespace janus;

extern "C" int janus_grouped_gemm(janus_ctx* ctx, const float* A, const float* B, float* C,
                                  const int32_t* row_off, int32_t n_groups, int64_t M, int32_t K, int32_t N,
                                  int32_t trans_b, void* stream) {
  if (!ctx || (M > 0 && (!A || !C)) || !B || !row_off || n_groups < 1 || n_groups > 1024 || M < 0 || M > INT32_MAX ||
      K <= 0 || K % GBK || N <= 0 || N % 64)
    return JANUS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int mt = max_rows_tiles(M, n_groups);
  Carver cv(nullptr);
  cv.take<RowsTile>(mt);
  cv.take<int>(1);
  int rc = ensure(ctx->aux, cv.size());
  if (rc) return rc;
  Carver c2(ctx->aux.ptr);
  RowsTile* tiles = c2.take<RowsTile>(mt);
  int* nt = c2.take<int>(1);
  grouped_rows(st, A, B, C, row_off, n_groups, K, N, trans_b, tiles, nt, mt);
  JANUS_HIP_TRY(hipGetLastError());
  return JANUS_OK;
}

// Fixed scratch of janus_grouped_gemm_noalloc: the tile table and its count.
// One copy per device, allocated with the library's code object on that
// device and held until the process ends; host code uses only the address
// returned by hipGetSymbolAddress for the current device, never the symbol.
constexpr size_t kNoAllocScratchBytes = size_t(4) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Address of the current device's scratch, looked up once per device.
int noalloc_scratch(void** out) {
  int dev = 0;
  JANUS_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return JANUS_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    JANUS_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return JANUS_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return JANUS_OK;
}

}  // namespace

// Largest tile table the fixed scratch holds (tiles first, then the count).
static int noalloc_max_tiles() {
  return (int)((kNoAllocScratchBytes - 256) / sizeof(RowsTile));
}

extern "C" int janus_grouped_gemm_noalloc(const float* A, const float* B, float* C, const int32_t* row_off,
                                          int32_t n_groups, int64_t M, int32_t K, int32_t N, int32_t trans_b,
                                          void* stream) {
  if ((M > 0 && (!A || !C)) || !B || !row_off || n_groups < 1 || n_groups > 1024 || M < 0 || M > INT32_MAX ||
      K <= 0 || K % GBK || N <= 0 || N % 64)
    return JANUS_EINVAL;
  const int mt = max_rows_tiles(M, n_groups);
  if (mt > noalloc_max_tiles()) return JANUS_ENOMEM;
  void* base = nullptr;
  int rc = noalloc_scratch(&base);
  if (rc) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  Carver cv(base);
  RowsTile* tiles = cv.take<RowsTile>(mt);
  int* nt = cv.take<int>(1);
  if (cv.size() > kNoAllocScratchBytes) return JANUS_ENOMEM;
  // the table kernel rewrites the count and every tile that the launch reads (a launch
  // without a table reads neither), so nothing left by an earlier call is used
  grouped_rows(st, A, B, C, row_off, n_groups, K, N, trans_b, tiles, nt, mt);
  JANUS_HIP_TRY(hipGetLastError());
  return JANUS_OK;
}

extern "C" int32_t janus_wgrad_chunk_rows(int64_t M, int32_t P, int32_t Q) {
  if (M < 0 || M > INT32_MAX || P <= 0 || Q <= 0) return JANUS_EINVAL;
  return wgrad_chunk_rows(M, P, Q);
}

extern "C" int janus_grouped_wgrad(janus_ctx* ctx, const float* A, const float* B, float* G,
                                   const int32_t* row_off, int32_t n_groups, int64_t M, int32_t P, int32_t Q,
                                   void* stream) {
  if (!ctx || (M > 0 && (!A || !B)) || !G || !row_off || n_groups < 1 || n_groups > 1024 || M < 0 || M > INT32_MAX ||
      P <= 0 || P % 4 || Q <= 0 || Q % 4)
    return JANUS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int kc = wgrad_chunk_rows(M, P, Q);
  const int mc = max_wchunks(M, n_groups, kc);
  Carver cv(nullptr);
  cv.take<WChunk>(mc);
  cv.take<int>(1);
  cv.take<int>(n_groups + 1);
  cv.take<float>((size_t)mc * P * Q);
  int rc = ensure(ctx->aux, cv.size());
  if (rc) return rc;
  Carver c2(ctx->aux.ptr);
  WChunk* chunks = c2.take<WChunk>(mc);
  int* nc = c2.take<int>(1);
  int* first = c2.take<int>(n_groups + 1);
  float* partial = c2.take<float>((size_t)mc * P * Q);
  build_tables(st, tables_of(row_off, n_groups).wgrad_chunks(kc, chunks, nc, first));
  launch_wgrad(std::true_type{}, st, LoadPlain{A, P}, LoadPlain{B, Q}, P, Q, chunks, nc, first, mc, n_groups, partial, G, 0);
  JANUS_HIP_TRY(hipGetLastError());
  return JANUS_OK;
}
