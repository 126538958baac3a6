// The steps on either side of the solve: building the dense matrix from an edge
// list (Section III: the program writes the input edge list into the adjacency
// matrix, both orientations unless the graph is directed), and reading paths
// back out of pred (Algorithm 1 records pred[v] = u for the edge that last
// improved dist[v]).
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>

#include "sssp.h"

namespace sssp {
int set_error(int code, const char* msg);
}

namespace {

constexpr int32_t kInf = 0x7fffffff;

int err(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return sssp::set_error(code, buf);
}

// W[i][j] = 0 on the diagonal, INT32_MAX (no edge) elsewhere; *bad = 0.  Bound by
// the writes: a workgroup takes one segment of a row, kFillSeg entries that start on
// a cache line whatever the row's alignment, as 16-byte stores (entries outside the
// row are left alone: there may be gaps between rows).  4-byte stores of a thread an entry
// took 232 us of a call's 291 at n=16000 (4.4 TB/s) and no less than 318 at n=16001;
// now 245 and 247 us a call, 1257 -> 1203 at n=40000 (5.5 TB/s).  Grids of 1024 to
// 8192 workgroups that loop took 263 to 285 us and, at n=16001, 315 to 372.
constexpr int kFillThreads = 256;
constexpr int kFillSeg = 4096;
constexpr int kLineEntries = 32;
constexpr int64_t kStreamBytes = 256ll << 20;  // what the memory-side cache holds

typedef int32_t quad __attribute__((ext_vector_type(4)));

template <bool Stream>
__global__ __launch_bounds__(kFillThreads) void k_fill_empty(int32_t* __restrict__ W, int64_t ld, int32_t n,
                                                             int32_t segs, unsigned long long* __restrict__ bad) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *bad = 0;
    for (int64_t t = blockIdx.x; t < (int64_t)segs * n; t += gridDim.x) {
        const int64_t i = t / segs;
        int32_t* row = W + i * ld;
        const int64_t off = ((uintptr_t)row >> 2) & (kLineEntries - 1);
        const int64_t j0 = (t - i * segs) * kFillSeg - off, j1 = j0 + kFillSeg < n ? j0 + kFillSeg : n;
        for (int64_t j = j0 + 4 * (int64_t)threadIdx.x; j < j1; j += 4 * kFillThreads) {
            quad v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = j + c == i ? 0 : kInf;
            if (j >= 0 && j + 4 <= n) {
                quad* q = reinterpret_cast<quad*>(row + j);
                if (Stream)
                    __builtin_nontemporal_store(v, q);
                else
                    *q = v;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (j + c >= 0 && j + c < n) row[j + c] = v[c];
            }
        }
    }
}

// Scatter the edges with an atomic minimum, so a duplicated edge keeps its
// smallest weight; a self-loop leaves the diagonal at 0.  Edges with an
// endpoint outside [0, n) or a weight outside [0, INT32_MAX) are skipped and
// counted in *bad.
__global__ void k_scatter_edges(const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                const int32_t* __restrict__ ew, int64_t m, int32_t n, int32_t directed,
                                int32_t* __restrict__ W, int64_t ld, unsigned long long* __restrict__ bad) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t u = eu[e], v = ev[e], w = ew[e];
        if (u < 0 || u >= n || v < 0 || v >= n || w < 0 || w == kInf) {
            atomicAdd(bad, 1ull);
            continue;
        }
        if (u == v) continue;
        atomicMin(&W[(int64_t)u * ld + v], w);
        if (!directed) atomicMin(&W[(int64_t)v * ld + u], w);
    }
}

// Pointer jumping over the pred forest: after the last pass hops[v] is the
// number of edges on v's pred chain to the source (0 at the source, -1 when v
// is unreachable).  A word holds (ancestor, hops so far).
struct Jump {
    int32_t anc, hop;
};

__device__ __forceinline__ Jump jump_start(const int32_t* __restrict__ pred, const int32_t* __restrict__ dist,
                                           int32_t v) {
    const int32_t p = pred[v];
    const bool reach = dist[v] != kInf;
    return Jump{reach ? p : -1, reach ? (p >= 0 ? 1 : 0) : -1};
}

// Each pass follows 2^log2_links links of the one before (of pred, in the first).
// Bound by launches and, in a pass, by the chain of reads: passes of one doubling
// took 4.7 us each at n=40000, 18 of them, though few chains of shortest path trees
// go beyond the first 32 links; now 8 us, then 3 passes of 4.
__global__ void k_hops_first(const int32_t* __restrict__ pred, const int32_t* __restrict__ dist, int32_t n,
                             int32_t log2_links, Jump* __restrict__ out) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        Jump x = jump_start(pred, dist, v);
        for (int32_t k = 1; k < 1 << log2_links && x.anc >= 0 && x.anc < n; ++k) {
            const Jump y = jump_start(pred, dist, x.anc);
            x = Jump{y.anc, (int32_t)((uint32_t)x.hop + (uint32_t)y.hop)};
        }
        out[v] = x;
    }
}

// Following more links in a pass reads more words for the same doublings: on large
// graphs that counts for more than launches.  One doubling a pass, two words each,
// and passes of 5, then 2 and of 1, then 2 doublings: n=10^6 a random tree 203, 195
// and 146 us, a single chain 523, 787 and 348; n=100000 97, 85 and 66; n=40000 79 and,
// with 5, then 4, 42 us.
constexpr int kHopsFirst = 5, kHopsFirstWide = 1;
constexpr int kHopsStep = 4, kHopsStepWide = 2;
constexpr int32_t kHopsWideN = 65536;

// hops (if given) takes the result instead of out.
__global__ void k_hops_step(const Jump* __restrict__ in, int32_t n, int32_t log2_links, Jump* __restrict__ out,
                            int32_t* __restrict__ hops) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        Jump x = in[v];
        for (int32_t k = 1; k < 1 << log2_links && x.anc >= 0 && x.anc < n; ++k) {
            const Jump y = in[x.anc];
            x = Jump{y.anc, (int32_t)((uint32_t)x.hop + (uint32_t)y.hop)};
        }
        if (hops)
            hops[v] = x.hop;
        else
            out[v] = x;
    }
}

// One thread per target: walk pred back from the target and write the path
// source ... target into out[off[i] .. off[i] + hops[t]].
__global__ void k_paths(const int32_t* __restrict__ pred, const int32_t* __restrict__ hops, int32_t n,
                        const int32_t* __restrict__ targets, int32_t count, const int64_t* __restrict__ off,
                        int32_t* __restrict__ out) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        int32_t v = targets[i];
        if (v < 0 || v >= n) continue;
        const int32_t h = hops[v];
        if (h < 0) continue;
        for (int32_t k = h; k >= 0 && v >= 0 && v < n; --k) {
            out[off[i] + k] = v;
            v = pred[v];
        }
    }
}

}  // namespace

extern "C" {

int sssp_edges_to_dense(const int32_t* eu, const int32_t* ev, const int32_t* ew, int64_t m, int32_t n,
                        int32_t directed, int32_t* W, int64_t ld, int64_t* bad_edges, void* stream) {
    if (!W || n < 1 || ld < n || m < 0 || (m > 0 && (!eu || !ev || !ew)))
        return err(SSSP_EINVAL, "bad arguments (n=%d ld=%lld m=%lld)", n, (long long)ld, (long long)m);
    hipStream_t s = (hipStream_t)stream;
    unsigned long long* d_bad = nullptr;
    hipError_t e = hipMallocAsync((void**)&d_bad, sizeof(unsigned long long), s);
    if (e != hipSuccess) return err(SSSP_ENOMEM, "hipMallocAsync: %s", hipGetErrorString(e));
    const int32_t segs = (int32_t)(((int64_t)n + kLineEntries - 1 + kFillSeg - 1) / kFillSeg);
    const int64_t all = (int64_t)n * segs;
    // a matrix larger than the memory-side cache streams past it (n=16001 247 us
    // against 271; n=4000, which stays in it, 66 us against 58)
    const bool stream_past = (int64_t)n * n * (int64_t)sizeof(int32_t) > kStreamBytes;
    hipLaunchKernelGGL(stream_past ? k_fill_empty<true> : k_fill_empty<false>,
                       dim3((unsigned)(all < 0x7fffff ? all : 0x7fffff)), dim3(kFillThreads), 0, s, W, ld, n, segs,
                       d_bad);
    e = hipGetLastError();
    if (e == hipSuccess && m > 0) {
        const int64_t blocks = (m + 255) / 256 < 8192 ? (m + 255) / 256 : 8192;
        hipLaunchKernelGGL(k_scatter_edges, dim3((unsigned)blocks), dim3(256), 0, s, eu, ev, ew, m, n, directed, W, ld,
                           d_bad);
        e = hipGetLastError();
    }
    unsigned long long bad = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&bad, d_bad, sizeof bad, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFreeAsync(d_bad, s);
    if (e != hipSuccess) return err(SSSP_EDEVICE, "edge list conversion: %s", hipGetErrorString(e));
    if (bad_edges) *bad_edges = (int64_t)bad;
    return SSSP_OK;
}

int sssp_hops(const int32_t* pred, const int32_t* dist, int32_t n, int32_t* hops, void* stream) {
    if (!pred || !dist || !hops || n < 1) return err(SSSP_EINVAL, "bad arguments");
    hipStream_t s = (hipStream_t)stream;
    Jump* buf = nullptr;
    hipError_t e = hipMallocAsync((void**)&buf, 2 * sizeof(Jump) * (size_t)n, s);
    if (e != hipSuccess) return err(SSSP_ENOMEM, "hipMallocAsync: %s", hipGetErrorString(e));
    const unsigned blocks = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    // ceil(log2 n) + 1 doublings reach the root of every chain
    int left = 1;
    while ((1ll << (left - 1)) < n) ++left;
    // the first pass leaves the last one something: that writes hops, and hops may be pred
    const int first = n < kHopsWideN ? kHopsFirst : kHopsFirstWide;
    int now = left > first ? first : left - 1;
    hipLaunchKernelGGL(k_hops_first, dim3(blocks), dim3(256), 0, s, pred, dist, n, now, buf);
    Jump *in = buf, *out = buf + n;
    const int each = n < kHopsWideN ? kHopsStep : kHopsStepWide;
    while ((left -= now) > 0) {
        now = left < each ? left : each;
        hipLaunchKernelGGL(k_hops_step, dim3(blocks), dim3(256), 0, s, in, n, now, out, left == now ? hops : nullptr);
        Jump* t = in;
        in = out;
        out = t;
    }
    e = hipGetLastError();
    (void)hipFreeAsync(buf, s);
    if (e != hipSuccess) return err(SSSP_EDEVICE, "hops: %s", hipGetErrorString(e));
    return SSSP_OK;
}

int sssp_paths(const int32_t* pred, const int32_t* hops, int32_t n, const int32_t* targets, int32_t count,
               const int64_t* offsets, int32_t* out, void* stream) {
    if (!pred || !hops || n < 1 || count < 0 || (count > 0 && (!targets || !offsets || !out)))
        return err(SSSP_EINVAL, "bad arguments");
    if (count == 0) return SSSP_OK;
    const unsigned blocks = (unsigned)((count + 255) / 256 < 4096 ? (count + 255) / 256 : 4096);
    hipLaunchKernelGGL(k_paths, dim3(blocks), dim3(256), 0, (hipStream_t)stream, pred, hops, n, targets, count,
                       offsets, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return err(SSSP_EDEVICE, "paths: %s", hipGetErrorString(e));
    return SSSP_OK;
}

}  // extern "C"
