// Transfer stage of the layer-wise pipeline (Section 3.4): many small copies
// in one launch (gfx950).
//
// A request made of documents brings a few hundred cache fragments per layer,
// each a few hundred KB, from wherever the store put them.  A copy on the DMA
// engines costs about 9 us beside its bytes, and they run one after the other:
// 360 copies of 364 KB took 5.7 ms (23 GB/s) where PCIe allows 2.3 ms; with
// this kernel the layer takes 2.64 ms.  A
// few workgroups read the fragments straight from pinned host memory over
// PCIe and write them to their rows: 57 GB/s with 32 workgroups of 256
// threads, 52 with 16 of 1,024, 46 with 8 of those, 8 GB/s per CU at most
// (the reads a CU can have outstanding).  The kernel may run beside a layer's
// attention, whose workgroups need a CU each, so it takes 16 CUs and not 32.
// Beside the attention of 124,256-row layers, per layer: fragments of 200 KB
// 35.3 -> 21.3 ms, 512 KB 20.4 -> 17.5, 1,000 KB 17.7 -> 17.5 (15.5 without
// any copies), so larger ones stay on the DMA engines.
// Fragments in device memory are copied the same way over all CUs: one launch
// instead of one of 1.6 us on the GPU and 2.5 on the host per fragment, up to
// the size (api.cpp) from which the runtime's faster copy makes up for that.
#include "kvc_internal.h"
#include "bf16_util.h"

namespace kvc {
namespace {

constexpr int kThreads = 1024;
constexpr int kUnits = 4;                        // 16-byte loads per thread in flight
constexpr uint32_t kTile = kThreads * kUnits;    // 16-byte units per tile (64 KB)
constexpr uint32_t kHostWorkgroups = 16;
constexpr uint32_t kDeviceWorkgroups = 2048;

// Tiles never cross entries; every workgroup walks tiles of the whole list.
__global__ __launch_bounds__(kThreads) void copy_list_kernel(const CopyList L) {
  const uint32_t tiles = L.end_tile[L.n - 1];
  for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    int lo = 0, hi = L.n - 1;  // the first entry whose end lies past the tile
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (L.end_tile[mid] > tile) hi = mid;
      else lo = mid + 1;
    }
    const uint64_t u0 = (uint64_t)(tile - (lo ? L.end_tile[lo - 1] : 0u)) * kTile + threadIdx.x;
    const uint64_t units = L.units[lo];
    const uint4* src = static_cast<const uint4*>(L.src[lo]);
    uint4* dst = static_cast<uint4*>(L.dst[lo]);
    uint4 v[kUnits];
#pragma unroll
    for (int i = 0; i < kUnits; ++i) {
      const uint64_t u = u0 + (uint64_t)i * kThreads;
      if (u < units) v[i] = load_nt(src + u);
    }
#pragma unroll
    for (int i = 0; i < kUnits; ++i) {
      const uint64_t u = u0 + (uint64_t)i * kThreads;
      if (u < units) dst[u] = v[i];
    }
  }
}

}  // namespace

bool copy_list_add(CopyList* L, void* dst, const void* src, size_t bytes) {
  const uint64_t units = bytes / 16, before = L->n ? L->end_tile[L->n - 1] : 0;
  const uint64_t end = before + (units + kTile - 1) / kTile;
  if (L->n == CopyList::kMax || units > UINT32_MAX || end > UINT32_MAX - kDeviceWorkgroups) return false;
  L->src[L->n] = src;
  L->dst[L->n] = dst;
  L->units[L->n] = (uint32_t)units;
  L->end_tile[L->n++] = (uint32_t)end;
  return true;
}

hipError_t launch_copy_list(const CopyList& L, bool host, hipStream_t s) {
  if (L.n == 0) return hipSuccess;
  const uint32_t grid = std::min(L.end_tile[L.n - 1], host ? kHostWorkgroups : kDeviceWorkgroups);
  hipLaunchKernelGGL(copy_list_kernel, dim3(grid), dim3(kThreads), 0, s, L);
  return hipGetLastError();
}

}  // namespace kvc
