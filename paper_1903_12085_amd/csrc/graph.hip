// Device graph: CSR upload and validation, static minima
// (equations crit:instatic / crit:outstatic need min in- and out-edge weight
// per vertex, computed once in O(m), Section 3; the implementation section
// computes the minimum in-edge weight with an atomic minimum per edge), and
// the per-row weight sort and the reverse adjacency (CSC), both built lazily
// for the dynamic criteria.
#include <algorithm>
#include <mutex>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <rocprim/rocprim.hpp>

#include "common.h"
#include "graph.h"

// ---------------------------------------------------------------------------
// error reporting

static thread_local char g_err[512] = "";

int sssp_set_error(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

extern "C" const char *sssp_last_error(void) { return g_err; }

// ---------------------------------------------------------------------------
// kernels

// What creation learns about a graph, spread over kShards slots on lines of their own (same-address
// atomics of many blocks serialise).
struct CreateInfo {
    struct alignas(128) Slot {
        unsigned long long sum_w;   // sum of the weights
        unsigned long long wmax;    // edges of weight 2^32 - 1
        unsigned int max_deg;       // longest row
    } s[kShards];
    unsigned int bad;               // malformed CSR: 1 = rows, 2 = ends, 4 = targets
};

// One pass over the input: rows to 32 bits, edges to (target, weight) in input order, the weights'
// sum and the edges of weight 2^32 - 1, and the checks row_ptr[0] == 0, monotone rows,
// row_ptr[n] == m, col < n. Later kernels do nothing once a check has failed.
__global__ __launch_bounds__(256) void k_load_csr(uint32_t n, uint64_t m, const uint64_t *__restrict__ rp64,
                                                  const uint32_t *__restrict__ col, const uint32_t *__restrict__ w,
                                                  uint32_t *__restrict__ rp, uint2 *__restrict__ edges, CreateInfo *info) {
    __shared__ unsigned long long sh[8 * 4];
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned int bad = 0;
    for (uint64_t v = t0; v <= n; v += stride) {
        const uint64_t x = rp64[v];
        if (v < n && rp64[v + 1] < x) bad |= 1u;
        if ((v == 0 && x != 0) || (v == n && x != m)) bad |= 2u;
        rp[v] = (uint32_t)x;
    }
    unsigned long long r[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // [0] weights, [1] edges of weight 2^32 - 1
    for (uint64_t e = t0; e < m; e += stride) {
        const uint2 ed = make_uint2(col[e], w[e]);
        if (ed.x >= n) bad |= 4u;
        r[0] += ed.y;
        r[1] += ed.y == INF32 ? 1u : 0u;
        edges[e] = ed;
    }
    if (bad) atomicOr(&info->bad, bad);
    block_reduce<4, 3u, 0u>(r, sh);
    if (threadIdx.x == 0) {
        CreateInfo::Slot &s = info->s[blockIdx.x % kShards];
        if (r[0]) atomicAdd(&s.sum_w, r[0]);
        if (r[1]) atomicAdd(&s.wmax, r[1]);
    }
}

// key = (target << 32) | weight for the reverse adjacency; payload = source.
__global__ void k_col_keys(uint64_t m, const uint2 *__restrict__ edges, const uint32_t *__restrict__ rp,
                           uint32_t n, unsigned long long *__restrict__ key, uint32_t *__restrict__ src) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
         e += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t lo = 0, hi = n - 1;
        while (lo < hi) {
            uint32_t mid = lo + (hi - lo + 1) / 2;
            if (rp[mid] <= e) lo = mid; else hi = mid - 1;
        }
        uint2 ed = edges[e];
        key[e] = ((unsigned long long)ed.x << 32) | ed.y;
        src[e] = lo;
    }
}

__global__ void k_pack_edges(uint64_t m, const unsigned long long *__restrict__ key,
                             const uint32_t *__restrict__ val, uint2 *__restrict__ out) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
         e += (uint64_t)gridDim.x * blockDim.x)
        out[e] = make_uint2(val[e], (uint32_t)(key[e] & 0xFFFFFFFFull));
}

// minOut = the lightest edge of each row (rows in input order); minIn reset to INF.
// A wavefront takes 64 consecutive rows, whose edges are contiguous: it reads
// them 64 at a time (coalesced), finds each edge's row among the 64 by a
// binary search over the row starts held one per lane, and folds the weight
// into that row's minimum in LDS.
__global__ __launch_bounds__(256) void k_min_out(uint32_t n, const uint32_t *__restrict__ rp,
                                                 const uint2 *__restrict__ edges, uint2 *__restrict__ vmin,
                                                 CreateInfo *info) {
    if (info->bad) return;  // grid-uniform
    __shared__ uint32_t smin[256];
    uint32_t dmax = 0;
    const uint32_t lane = threadIdx.x & 63;
    uint32_t *wmin = smin + (threadIdx.x & ~63u);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63u); base < n; base += stride) {
        const uint64_t v = base + lane;  // base is wavefront-uniform
        const uint32_t rs = v < n ? rp[v] : rp[n];  // this lane's row start (rows past n are empty)
        const uint32_t e0 = (uint32_t)__shfl((int)rs, 0, 64);
        const uint32_t e1 = rp[base + 64 < n ? base + 64 : n];
        const uint32_t next = (uint32_t)__shfl_down((int)rs, 1, 64);
        dmax = max(dmax, (lane == 63 ? e1 : next) - rs);  // rows past n start at e1
        wmin[lane] = INF32;
        __builtin_amdgcn_wave_barrier();
        for (uint32_t k = e0 + lane; __ballot(k < e1); k += 64) {  // wavefront-uniform
            const bool in = k < e1;
            const uint32_t w = in ? edges[k].y : INF32;
            int lo = 0;  // last row of the window whose start is <= k (every lane shuffles)
#pragma unroll
            for (int st = 32; st > 0; st >>= 1) {
                const uint32_t r = (uint32_t)__shfl((int)rs, lo + st, 64);
                if (r <= k) lo += st;
            }
            if (in) atomicMin(&wmin[lo], w);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (v < n) vmin[v] = make_uint2(INF32, wmin[lane]);
        __builtin_amdgcn_wave_barrier();
    }
    for (int o = 32; o > 0; o >>= 1) dmax = max(dmax, (uint32_t)__shfl_xor((int)dmax, o, 64));
    unsigned int *slot = &info->s[blockIdx.x % kShards].max_deg;
    if (lane == 0 && dmax > *slot) atomicMax(slot, dmax);
}

// key = (row << 32) | weight and payload = target of every edge, for the row
// sort; the row by binary search in row_ptr.
__global__ void k_row_keys_e(uint32_t n, uint64_t m, const uint32_t *__restrict__ rp, const uint2 *__restrict__ edges,
                             unsigned long long *__restrict__ key, uint32_t *__restrict__ val) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
         e += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t lo = 0, hi = n - 1;
        while (lo < hi) {
            uint32_t mid = lo + (hi - lo + 1) / 2;
            if (rp[mid] <= e) lo = mid; else hi = mid - 1;
        }
        const uint2 ed = edges[e];
        key[e] = ((unsigned long long)lo << 32) | ed.y;
        val[e] = ed.x;
    }
}

// Per edge (u, v): emin = minOut of v (relax folds the next OUT-STATIC threshold from the edge's own
// position), and c(u, v) into minIn of v, by an atomic minimum where it is lower. Both come from one
// random 8-byte load of v's minima, four edges' loads issued together: bound by the rate of random
// lines, 1.2 ms for 2^26 edges over 2^22 vertices (with a pass for each minimum 2.4 ms).
__global__ __launch_bounds__(256) void k_edge_minima(uint64_t m, const uint2 *__restrict__ edges, uint2 *vmin,
                                                     uint32_t *__restrict__ emin, const CreateInfo *info) {
    if (info->bad) return;  // grid-uniform
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e0 < m; e0 += 4 * stride) {
        uint2 ed[4], mm[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (e0 + j * stride < m) ed[j] = edges[e0 + j * stride];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (e0 + j * stride < m) mm[j] = vmin[ed[j].x];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (e0 + j * stride < m) {
                emin[e0 + j * stride] = mm[j].y;
                if (ed[j].y < mm[j].x) atomicMin(&vmin[ed[j].x].x, ed[j].y);
            }
    }
}

// After the rows were sorted: emin[e] = minOut of edge e's target: relax folds the next OUT-STATIC threshold
// from the edge's own row position, with no load that waits for the atomic.
__global__ void k_emin(uint64_t m, const uint2 *__restrict__ edges, const uint2 *__restrict__ vmin,
                       uint32_t *__restrict__ emin) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (uint64_t)gridDim.x * blockDim.x)
        emin[e] = vmin[edges[e].x].y;
}

// in_ptr[v] = first index whose sorted key has target >= v.
__global__ void k_in_ptr(uint32_t n, uint64_t m, const unsigned long long *__restrict__ key,
                         uint32_t *__restrict__ ip) {
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v <= n;
         v += (uint64_t)gridDim.x * blockDim.x) {
        unsigned long long target = (unsigned long long)v << 32;
        uint64_t lo = 0, hi = m;
        while (lo < hi) {
            uint64_t mid = (lo + hi) / 2;
            if (key[mid] < target) lo = mid + 1; else hi = mid;
        }
        ip[v] = (uint32_t)lo;
    }
}

static inline int grid_for(uint64_t items, int block = 256, int cap = 8192) {
    uint64_t g = (items + block - 1) / block;
    if (g < 1) g = 1;
    if (g > (uint64_t)cap) g = cap;
    return (int)g;
}

static int bits_for(uint32_t n) {
    int b = 1;
    while (b < 32 && (1ull << b) < n) ++b;
    return b;
}

// Sort (key, value) pairs with rocPRIM's device radix sort, in place via a
// second buffer pair; `end_bit` bounds the key width.
static int radix_sort(unsigned long long *&k0, unsigned long long *&k1, uint32_t *&v0, uint32_t *&v1,
                      uint64_t m, int end_bit, hipStream_t s) {
    size_t tmp_bytes = 0;
    if (rocprim::radix_sort_pairs(nullptr, tmp_bytes, k0, k1, v0, v1, (size_t)m, 0, end_bit, s) != hipSuccess)
        return sssp_set_error(SSSP_ERR_DEVICE, "radix_sort_pairs size query failed");
    void *tmp = nullptr;
    HIP_OK(sssp_malloc(&tmp, tmp_bytes ? tmp_bytes : 1));
    hipError_t e = rocprim::radix_sort_pairs(tmp, tmp_bytes, k0, k1, v0, v1, (size_t)m, 0, end_bit, s);
    hipError_t e2 = hipStreamSynchronize(s);
    sssp_free(tmp);
    if (e != hipSuccess || e2 != hipSuccess)
        return sssp_set_error(SSSP_ERR_DEVICE, "radix_sort_pairs failed: %s", hipGetErrorString(e != hipSuccess ? e : e2));
    unsigned long long *tk = k0; k0 = k1; k1 = tk;  // sorted data now in k0 / v0
    uint32_t *tv = v0; v0 = v1; v1 = tv;
    return SSSP_OK;
}

// ---------------------------------------------------------------------------
// host API

// One freed graph allocation per device is kept for the next graph: hipFree of a block of more than
// 64 MiB takes 0.33 to 8 ms (smaller ones 12 us: the runtime keeps those itself), as much as the rest
// of a creation or more. At most kKeepMax bytes; given back when an allocation fails, and by
// sssp_graph_destroy(NULL). Every call on a graph has finished its device work when it returns, so a
// block is idle here. 2 GiB hold a graph of 2^27 edges, and are 0.7 % of the memory; with 512 MiB the
// creation and release of one of 2^26 edges took 4 or 33 ms, by the process, now 1.8.
constexpr uint64_t kKeepMin = 64ull << 20, kKeepMax = 2ull << 30;
constexpr int kKeepDevices = 64;
static std::mutex g_keep_mu;
static struct { void *p; uint64_t bytes; } g_keep[kKeepDevices];

static hipError_t block_alloc(int dev, uint64_t bytes, void **p, uint64_t *got) {
    if (dev < kKeepDevices && bytes > kKeepMin) {
        std::lock_guard<std::mutex> lock(g_keep_mu);
        auto &k = g_keep[dev];
        if (k.p && k.bytes >= bytes && k.bytes / 2 <= bytes) {
            *p = k.p;
            *got = k.bytes;
            k.p = nullptr;
            return hipSuccess;
        }
    }
    *got = bytes;
    return sssp_malloc_bytes(p, bytes);
}

static void block_free(int dev, void *p, uint64_t bytes) {
    if (p && dev < kKeepDevices && bytes > kKeepMin && bytes <= kKeepMax) {
        std::lock_guard<std::mutex> lock(g_keep_mu);
        std::swap(p, g_keep[dev].p);  // the block kept so far goes
        g_keep[dev].bytes = bytes;
    }
    sssp_free(p);
}

static void blocks_give_back() {
    std::lock_guard<std::mutex> lock(g_keep_mu);
    for (auto &k : g_keep) {
        sssp_free(k.p);
        k.p = nullptr;
    }
}

hipError_t sssp_malloc_bytes(void **p, uint64_t bytes) {
    hipError_t e = hipMalloc(p, bytes ? bytes : 1);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    blocks_give_back();
    e = hipMalloc(p, bytes ? bytes : 1);
    if (e == hipErrorOutOfMemory) (void)hipGetLastError();  // reported here, not by the next launch
    return e;
}

static uint64_t up256(uint64_t x) { return (x + 255) & ~255ull; }

// Everything is queued on the stream and read back once: the arrays lie in one allocation, and
// kernels that would follow a malformed row or target see the check's verdict on the device.
static int create_impl(uint32_t n, uint64_t m, const uint64_t *row_ptr, const uint32_t *col,
                       const uint32_t *weight, int device_ptrs, hipStream_t s, sssp_graph *g) {
    const uint64_t o_edges = up256(sizeof(CreateInfo)), o_emin = up256(o_edges + m * sizeof(uint2)),
                   o_vmin = up256(o_emin + m * sizeof(uint32_t)), o_rp = up256(o_vmin + (uint64_t)n * sizeof(uint2)),
                   total = o_rp + (n + 1ull) * sizeof(uint32_t);
    HIP_OK(block_alloc(g->device, total, &g->base, &g->base_bytes));
    uint8_t *base = (uint8_t *)g->base;
    CreateInfo *info = (CreateInfo *)base;
    g->edges = (uint2 *)(base + o_edges);
    g->emin = (uint32_t *)(base + o_emin);
    g->vmin = (uint2 *)(base + o_vmin);
    g->rp = (uint32_t *)(base + o_rp);
    HIP_OK(hipMemsetAsync(info, 0, sizeof(CreateInfo), s));
    CallBuffer stage;  // host input on the device
    if (!device_ptrs) {
        const uint64_t o_col = up256((n + 1ull) * sizeof(uint64_t)), o_w = up256(o_col + m * sizeof(uint32_t));
        HIP_OK(sssp_malloc(&stage.p, o_w + m * sizeof(uint32_t)));
        uint8_t *st = (uint8_t *)stage.p;
        HIP_OK(hipMemcpyAsync(st, row_ptr, (n + 1ull) * sizeof(uint64_t), hipMemcpyHostToDevice, s));
        if (m) {
            HIP_OK(hipMemcpyAsync(st + o_col, col, m * sizeof(uint32_t), hipMemcpyHostToDevice, s));
            HIP_OK(hipMemcpyAsync(st + o_w, weight, m * sizeof(uint32_t), hipMemcpyHostToDevice, s));
        }
        row_ptr = (const uint64_t *)st;
        col = (const uint32_t *)(st + o_col);
        weight = (const uint32_t *)(st + o_w);
    }
    struct Events {
        hipEvent_t e[2] = {nullptr, nullptr};
        ~Events() {
            for (hipEvent_t x : e)
                if (x) (void)hipEventDestroy(x);
        }
    } ev;
    for (hipEvent_t &x : ev.e) HIP_OK(hipEventCreate(&x));
    HIP_OK(hipEventRecord(ev.e[0], s));
    hipLaunchKernelGGL(k_load_csr, dim3(grid_for(m > n ? m : n + 1ull, 256, 4096)), dim3(256), 0, s, n, m, row_ptr, col,
                       weight, g->rp, g->edges, info);
    hipLaunchKernelGGL(k_min_out, dim3(grid_for(n)), dim3(256), 0, s, n, g->rp, g->edges, g->vmin, info);
    if (m) hipLaunchKernelGGL(k_edge_minima, dim3(grid_for(m, 1024)), dim3(256), 0, s, m, g->edges, g->vmin, g->emin, info);
    HIP_OK(hipEventRecord(ev.e[1], s));
    HIP_OK(hipGetLastError());
    CreateInfo h;
    HIP_OK(hipMemcpyAsync(&h, info, sizeof h, hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    if (h.bad) return sssp_set_error(SSSP_ERR_INVALID, "malformed CSR (code %u)", h.bad);
    for (const CreateInfo::Slot &x : h.s) {
        g->sum_w += x.sum_w;
        g->wmax |= x.wmax != 0;
        g->max_deg = std::max(g->max_deg, x.max_deg);
    }
    float ms = 0;
    HIP_OK(hipEventElapsedTime(&ms, ev.e[0], ev.e[1]));
    g->precompute_ns = (uint64_t)(ms * 1e6);
    return SSSP_OK;
}

extern "C" int sssp_graph_create(uint32_t n, uint64_t m, const uint64_t *row_ptr, const uint32_t *col,
                                 const uint32_t *weight, int device_ptrs, void *hip_stream,
                                 sssp_graph **out) {
    if (!out) return sssp_set_error(SSSP_ERR_INVALID, "out is NULL");
    *out = nullptr;
    if (n == 0) return sssp_set_error(SSSP_ERR_INVALID, "n must be >= 1");
    if (!row_ptr || (m && (!col || !weight))) return sssp_set_error(SSSP_ERR_INVALID, "NULL CSR array");
    if (n >= (1u << 26) || m >= (1ull << 32))
        return sssp_set_error(SSSP_ERR_UNSUPPORTED, "graph too large (n=%u, m=%llu): need n < 2^26, m < 2^32",
                              n, (unsigned long long)m);
    if (!device_ptrs) {  // host-side validation
        if (row_ptr[0] != 0 || row_ptr[n] != m)
            return sssp_set_error(SSSP_ERR_INVALID, "row_ptr[0] must be 0 and row_ptr[n] must equal m");
        for (uint32_t v = 0; v < n; ++v)
            if (row_ptr[v + 1] < row_ptr[v]) return sssp_set_error(SSSP_ERR_INVALID, "row_ptr not monotone at %u", v);
        for (uint64_t e = 0; e < m; ++e)
            if (col[e] >= n) return sssp_set_error(SSSP_ERR_INVALID, "col[%llu] = %u >= n", (unsigned long long)e, col[e]);
    }
    sssp_graph *g = new (std::nothrow) sssp_graph();
    if (!g) return sssp_set_error(SSSP_ERR_OOM, "host allocation failed");
    g->n = n;
    g->m = m;
    g->stream = (hipStream_t)hip_stream;
    if (hipGetDevice(&g->device) != hipSuccess) { delete g; return sssp_set_error(SSSP_ERR_DEVICE, "no HIP device"); }
    int rc = create_impl(n, m, row_ptr, col, weight, device_ptrs, g->stream, g);
    if (rc != SSSP_OK) {
        // what was queued before the failure may write to the block, which the next graph can get
        if (g->base) (void)hipStreamSynchronize(g->stream);
        sssp_graph_destroy(g);
        return rc;
    }
    graph_default_cfg(g);
    *out = g;
    return SSSP_OK;
}

extern "C" int sssp_graph_destroy(sssp_graph *g) {
    if (!g) {
        blocks_give_back();
        return SSSP_OK;
    }
    block_free(g->device, g->base, g->base_bytes);  // rows, edges and minima
    sssp_free(g->ip); sssp_free(g->in_edges);
    sssp_free(g->res);
    sssp_free(g->one_fm);  // the one-workgroup scratch's other buffers go with solve_bufs_free
    solve_bufs_free(g);
    delete g;
    return SSSP_OK;
}

extern "C" int sssp_set_stream(sssp_graph *g, void *hip_stream) {
    if (!g) return sssp_set_error(SSSP_ERR_INVALID, "graph is NULL");
    g->stream = (hipStream_t)hip_stream;
    return SSSP_OK;
}

__global__ void k_split_minima(uint32_t n, const uint2 *__restrict__ vmin, uint32_t *mi, uint32_t *mo) {
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (uint64_t)gridDim.x * blockDim.x) {
        uint2 x = vmin[v];
        if (mi) mi[v] = x.x;
        if (mo) mo[v] = x.y;
    }
}

extern "C" int sssp_graph_minima(sssp_graph *g, uint32_t *min_in, uint32_t *min_out) {
    if (!g) return sssp_set_error(SSSP_ERR_INVALID, "graph is NULL");
    hipLaunchKernelGGL(k_split_minima, dim3(grid_for(g->n)), dim3(256), 0, g->stream, g->n, g->vmin, min_in, min_out);
    HIP_OK(hipGetLastError());
    HIP_OK(hipStreamSynchronize(g->stream));
    return SSSP_OK;
}

// Sorts each row of the CSR by weight, in place (the cursors of the dynamic
// criteria walk rows lightest first); emin follows the edges. Once per graph.
int graph_ensure_sorted(sssp_graph *g) {
    if (g->rows_sorted || g->m == 0) {
        g->rows_sorted = true;
        return SSSP_OK;
    }
    const uint64_t m = g->m;
    hipStream_t s = g->stream;
    unsigned long long *k0 = nullptr, *k1 = nullptr;
    uint32_t *v0 = nullptr, *v1 = nullptr;
    int rc = SSSP_OK;
#define TRY(call) do { hipError_t _e = (call); if (_e != hipSuccess) { \
        rc = sssp_set_error(_e == hipErrorOutOfMemory ? SSSP_ERR_OOM : SSSP_ERR_DEVICE, "%s: %s", #call, hipGetErrorString(_e)); goto done; } } while (0)
    TRY(sssp_malloc(&k0, m * sizeof(unsigned long long)));
    TRY(sssp_malloc(&k1, m * sizeof(unsigned long long)));
    TRY(sssp_malloc(&v0, m * sizeof(uint32_t)));
    TRY(sssp_malloc(&v1, m * sizeof(uint32_t)));
    hipLaunchKernelGGL(k_row_keys_e, dim3(grid_for(m)), dim3(256), 0, s, g->n, m, g->rp, g->edges, k0, v0);
    rc = radix_sort(k0, k1, v0, v1, m, 32 + bits_for(g->n), s);
    if (rc != SSSP_OK) goto done;
    hipLaunchKernelGGL(k_pack_edges, dim3(grid_for(m)), dim3(256), 0, s, m, k0, v0, g->edges);
    hipLaunchKernelGGL(k_emin, dim3(grid_for(m)), dim3(256), 0, s, m, g->edges, g->vmin, g->emin);
    TRY(hipGetLastError());
    TRY(hipStreamSynchronize(s));
    g->rows_sorted = true;
done:
#undef TRY
    sssp_free(k0); sssp_free(k1); sssp_free(v0); sssp_free(v1);
    return rc;
}

// Reverse adjacency with rows sorted by weight (for the dynamic IN terms).
int graph_ensure_csc(sssp_graph *g) {
    if (g->ip || g->m == 0) {
        if (!g->ip) {  // edgeless graph: all-zero in_ptr
            HIP_OK(sssp_malloc(&g->ip, (g->n + 1) * sizeof(uint32_t)));
            HIP_OK(hipMemsetAsync(g->ip, 0, (g->n + 1) * sizeof(uint32_t), g->stream));
            HIP_OK(sssp_malloc(&g->in_edges, sizeof(uint2)));
        }
        return SSSP_OK;
    }
    const uint64_t m = g->m;
    hipStream_t s = g->stream;
    unsigned long long *k0 = nullptr, *k1 = nullptr;
    uint32_t *v0 = nullptr, *v1 = nullptr;
    int rc = SSSP_OK;
    if (sssp_malloc(&k0, m * 8) != hipSuccess || sssp_malloc(&k1, m * 8) != hipSuccess ||
        sssp_malloc(&v0, m * 4) != hipSuccess || sssp_malloc(&v1, m * 4) != hipSuccess ||
        sssp_malloc(&g->ip, (g->n + 1) * sizeof(uint32_t)) != hipSuccess ||
        sssp_malloc(&g->in_edges, m * sizeof(uint2)) != hipSuccess) {
        rc = sssp_set_error(SSSP_ERR_OOM, "CSC allocation failed");
    } else {
        hipLaunchKernelGGL(k_col_keys, dim3(grid_for(m)), dim3(256), 0, s, m, g->edges, g->rp, g->n, k0, v0);
        rc = radix_sort(k0, k1, v0, v1, m, 32 + bits_for(g->n), s);
        if (rc == SSSP_OK) {
            hipLaunchKernelGGL(k_pack_edges, dim3(grid_for(m)), dim3(256), 0, s, m, k0, v0, g->in_edges);
            hipLaunchKernelGGL(k_in_ptr, dim3(grid_for(g->n + 1)), dim3(256), 0, s, g->n, m, k0, g->ip);
            if (hipStreamSynchronize(s) != hipSuccess) rc = sssp_set_error(SSSP_ERR_DEVICE, "CSC build failed");
        }
    }
    sssp_free(k0); sssp_free(k1); sssp_free(v0); sssp_free(v1);
    if (rc != SSSP_OK) {
        sssp_free(g->ip); sssp_free(g->in_edges);
        g->ip = nullptr; g->in_edges = nullptr;
    }
    return rc;
}
