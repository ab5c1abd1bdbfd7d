// Resident solver: the whole solve of one query in one cooperative launch, for
// sssp_solve and sssp_solve_noalloc with static criteria, for sssp_solve with SIMPLE
// ones, and for sssp_delta_step; and batches of queries, each by a team of workgroups
// (at the end of this file).
//
// W workgroups (a power of two) stay on the device for the whole solve. The
// vertices are cut into groups of K = 8 (16) consecutive ones; every group has an
// owner, one wavefront of one workgroup, that keeps in LDS the minima over the
// group's queued vertices of the IN-STATIC key d - minIn, of d and of d + minOut,
// and which of its vertices have settled. A phase (Section 3) then is, for a
// wavefront:
//   1. select   a lane per group: it is active if a relax of the last phase marked
//               it, or if its minima pass the phase's thresholds. Every other group
//               can neither settle a vertex nor change its minima.
//   2. identify a row of K lanes per active group: load the vertices' distances,
//               what the last phase delivered, and static minima; certify (eq.
//               crit:instatic, crit:outstatic), refresh the group's minima, cut
//               the out-edges of the settled vertices into segments of 16.
//   3. relax    a row of 16 lanes per segment: edge, target, 64-bit atomicMin into
//               the target's box; a mark on the target's group; fold into the next
//               minD / threshold.
//   4. combine  each workgroup publishes its next minD and threshold; reading
//               everybody's is both the reduction and the phase's only barrier.
// A phase must not see what the same phase delivers: a fast workgroup relaxes
// while a slow one still identifies. Each vertex therefore has two boxes, and
// each group two marks: relax of phase k writes those of parity k + 1, identify
// of phase k reads those of parity k and keeps the distance itself, which nobody
// else writes. Boxes and marks need no clearing: box values only fall, and a
// mark is the number of the phase it is for.
//
// Delta-stepping (Section 5) runs on the same structure, a round in the place of a
// phase: the first light round of a bucket relaxes the queued vertices inside the
// window, a further one those the last round lowered inside it (an owner sees that
// a box undercuts its distance), the heavy round those the bucket removed. The
// barrier carries whether anything was lowered inside the window, and after a
// heavy round the smallest queued distance.
//
// SIMPLE criteria (eq. crit:insimple, crit:outsimple): a vertex's term is the lightest edge of a
// sorted row whose other end has not settled; the vertex keeps that edge, its head. Certifying
// must not start before every head is current, and heads move when vertices settle, so a phase
// has a second barrier: refresh the heads, combine minD and T, certify, relax, meet. With it one
// box per vertex does; its top bit says settled. A relax marks its target also where the edge is
// the target's IN head. OUT heads would need the in-edges of all that settles, so they are
// checked lazily: a sum d + term seen before is a lower bound, and only a sum below the next T
// matters. Sums up to a guess, four times as far beyond the last T as that lay beyond its minD,
// are checked before the barrier; when T turns out larger, a further pass and barrier follow
// (1.5 passes a phase on a random graph with the guess one time as far, 1.1 with four times).
// R-MAT 20: 31.6 us a phase, 46.5 with the phase kernels; random, 1 M vertices of degree 16: 20.9
// and 38.2; 5000 of degree 9: 11.8 and 26.7. Half of a phase is the wait for the wavefront with
// the longest chain of loads in refresh.
//
// Skewed graphs (a row over kShareDeg edges): one workgroup's segments would
// hold up all, so its segments form one list, and rows past a quota, or longer
// than kHubEdges, become records in device memory that all workgroups relax. A
// second barrier, awaited after the own segments, tells how many there are.
//
// What bounds a phase is a chain of dependent round trips (mark, distance, edge,
// target, atomic and mark, barrier) and the skew between workgroups, not bytes:
// of the 10.4 us of a phase on the 2^22-vertex random graph about 2 are the
// barrier. The phase kernels need two launches a phase and about ten round
// trips: 24.9 us there, 15.9 on a 1023 x 997 grid (5.0 here), 25.9 on R-MAT 22
// (15.4 here), 18.0 on 16384 vertices of degree 8 (4.8 here).
//
// Values that several workgroups touch go through device-scope atomics, loads
// and stores; everything a workgroup wrote has completed when it publishes.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "common.h"
#include "graph.h"
#include "selector.h"
#include "words.h"

constexpr uint32_t kSegEdges = 16;     // edges per segment = lanes per row in relax
constexpr uint32_t kMaxJ = 4;          // slots per thread
constexpr uint32_t kWaveSegs = 64;     // segments a wavefront holds in LDS; further settled vertices stay pending
constexpr uint32_t kHubEdges = 1024;   // longer rows are cut by the whole wavefront
constexpr uint32_t kShareEdges = 256;  // edges of a shared record (more for a hub past kShareCap / 2 records)
constexpr uint32_t kShareCap = 1024;   // shared records per workgroup and phase
constexpr uint32_t kShareDeg = 128;    // graphs with a longer row share records (see `share` in ResArgs)
constexpr uint32_t kQuota = 64;        // segments a list takes in a phase before further rows are shared
constexpr uint32_t kResSpin = 1u << 21;  // polls of a wait (about 0.5 us each) before all give up

// Learned checkpoint solves.
struct ResLearn {
    unsigned long long sum[3];     // so far, at the last checkpoint: reached, settled before it, settled at checkpoints
    unsigned long long choice[2];  // the selector's choice, by checkpoint parity
    ResLearned out;
};

struct ResCtl {
    unsigned long long bar[team_words(kResMaxW)];     // see words.h
    unsigned int rank[16 * 32];                       // arrivals per XCD
    unsigned int error;
    unsigned int phases;
    ResLearn learn;
    unsigned int team;                                // 1 + the XCD whose workgroups form the team
};

struct ResArgs {
    const uint32_t *rp;
    const uint2 *edges;
    const uint2 *vmin;
    const uint32_t *emin;
    unsigned long long *dist;  // owners' distances; the output
    unsigned long long *box;   // per vertex, by phase parity: the lowest candidate relaxes delivered
    uint8_t *mark;       // by phase parity, W rows of mstride bytes: the phase tag each slot was last marked for
    unsigned long long *rec;    // W rows of kShareCap records (first edge and count, distance)
    unsigned long long *bar;    // the team's words (words.h)
    unsigned int *error;
    uint32_t n, src, wmax;
    uint32_t W, lgW;     // workgroups
    uint32_t lgWv;       // wavefronts per workgroup
    uint32_t wslots;     // slots per wavefront, a multiple of 64
    uint32_t mstride;    // slots per workgroup
    uint32_t quota;      // segments a wavefront keeps for itself in a phase
    uint32_t share;      // rows beyond the quota become records relaxed by all workgroups
    uint32_t lgK;        // vertices per group
    uint32_t max_phases; // a solve that takes more ends with an error
    uint32_t polls;      // of a wait for another workgroup
    unsigned long long delta;  // Delta-stepping: bucket width
    // SIMPLE criteria: the reverse adjacency and, per vertex, the lightest edge of each row whose other
    // end had not settled when the owner last looked, with its place in the row
    const uint32_t *ip;
    const uint2 *in_edges;
    uint2 *in_head, *out_head;
    uint32_t *in_cur, *out_cur;
    // learned checkpoint solves: per vertex the phase that settled it (from 1), the selector's weights
    // (and where in LDS a copy goes), mean edge weight, edges
    ResLearn *learn;
    uint32_t *sp;
    const float *mlp_w;
    double wm;
    uint64_t m;
    uint32_t mlp_lds;
};

__device__ __forceinline__ unsigned long long ld64(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_agent(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t umin32(uint32_t a, uint32_t b) { return a < b ? a : b; }
// Minimum over K = 8 or 16 consecutive lanes.
template <int K>
__device__ __forceinline__ unsigned long long row_min64(unsigned long long x) {
    x = umin64(x, dpp64<kDppQuadSwap1>(x));
    x = umin64(x, dpp64<kDppQuadSwap2>(x));
    x = umin64(x, dpp64<kDppHalfMirror>(x));
    return K == 16 ? umin64(x, dpp64<kDppMirror>(x)) : x;
}
template <int K>
__device__ __forceinline__ uint32_t row_min32(uint32_t x) {
    x = umin32(x, dpp32<kDppQuadSwap1>(x));
    x = umin32(x, dpp32<kDppQuadSwap2>(x));
    if (K >= 8) x = umin32(x, dpp32<kDppHalfMirror>(x));
    return K >= 16 ? umin32(x, dpp32<kDppMirror>(x)) : x;
}
// Minima of values that are INF64 or at least `base` (everything a phase keeps lies above its minD):
// the distances from the base mostly fit in 32 bits, which takes a quarter of the instructions.
__device__ __forceinline__ uint32_t rel32(unsigned long long x, unsigned long long base) {
    const unsigned long long r = x - base;
    return r >> 32 ? INF32 : (uint32_t)r;
}
template <int K>
__device__ __forceinline__ unsigned long long row_min_rel(unsigned long long x, unsigned long long base) {
    const uint32_t m = row_min32<K>(rel32(x, base));
    if (__ballot(m == INF32 && x != INF64)) return row_min64<K>(x);  // wavefront-uniform
    return m == INF32 ? INF64 : base + m;
}
__device__ __forceinline__ unsigned long long wave_min_rel(unsigned long long x, unsigned long long base) {
    const uint32_t r = row_min32<16>(rel32(x, base));
    const uint32_t m = umin32(umin32((uint32_t)__builtin_amdgcn_readlane((int)r, 0), (uint32_t)__builtin_amdgcn_readlane((int)r, 16)),
                              umin32((uint32_t)__builtin_amdgcn_readlane((int)r, 32), (uint32_t)__builtin_amdgcn_readlane((int)r, 48)));
    if (m != INF32) return base + m;
    return __ballot(x != INF64) ? wave_min64(x) : INF64;
}
// a / b rounded up, for any a (a row may hold nearly 2^32 edges)
__device__ __forceinline__ uint32_t ceil_div(uint32_t a, uint32_t b) { return a / b + (a % b != 0); }
__device__ __forceinline__ uint32_t phase_tag(uint32_t k) { return k % 255u + 1u; }

// Group g belongs to workgroup g mod W, there to wavefront (g / W) mod (wavefronts), as that
// wavefront's slot: neighbouring groups are spread over workgroups first, then over wavefronts.
__device__ __forceinline__ uint64_t mark_of(const ResArgs &a, uint32_t g) {
    const uint32_t t = g >> a.lgW;
    return (uint64_t)(g & (a.W - 1)) * a.mstride + (t & ((1u << a.lgWv) - 1u)) * a.wslots + (t >> a.lgWv);
}

__global__ void k_res_init(ResArgs a, ResCtl *ctl) {
    const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = t0; v < a.n; v += stride) {
        const unsigned long long x = v == a.src ? 0ull : INF64;
        a.dist[v] = x;
        a.box[2 * v] = x;
        a.box[2 * v + 1] = x;
        if (a.sp) a.sp[v] = 0;
    }
    const uint64_t src_mark = mark_of(a, a.src >> a.lgK);
    uint32_t *mw = reinterpret_cast<uint32_t *>(a.mark);
    for (uint64_t i = t0; i < (uint64_t)a.W * a.mstride / 2; i += stride)
        mw[i] = i == src_mark / 4 ? phase_tag(0) << (8 * (src_mark & 3)) : 0u;
    uint32_t *c = reinterpret_cast<uint32_t *>(ctl);
    for (uint64_t i = t0; i < sizeof(ResCtl) / 4; i += stride) c[i] = 0;
}

struct Seg {
    uint32_t e, len;
    unsigned long long d;
};

static size_t res_lds(uint32_t slots, int bs) {
    return (size_t)bs / 64 * kWaveSegs * sizeof(Seg) + (size_t)slots * (3 * 8 + 3 * 2);
}

__device__ __forceinline__ void wave_fence() {  // LDS values pass between lanes of one wavefront
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// SIMPLE criteria, instead of k_res_init: of the two words per vertex in `box` the first is the box,
// the second the weight of its IN head (all ones without one).
__global__ void k_res_init_simple(ResArgs a, ResCtl *ctl, int in_simple) {
    const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    const uint2 none = make_uint2(INF32, INF32);
    for (uint64_t v = t0; v < a.n; v += stride) {
        const unsigned long long x = v == a.src ? 0ull : INF64;
        a.dist[v] = x;
        const uint32_t o = a.rp[v];
        a.out_cur[v] = o;
        a.out_head[v] = o < a.rp[v + 1] ? a.edges[o] : none;
        uint2 h = none;
        if (in_simple) {
            const uint32_t i = a.ip[v];
            if (i < a.ip[v + 1]) h = a.in_edges[i];
            a.in_cur[v] = i;
            a.in_head[v] = h;
        }
        a.box[2 * v] = x;
        a.box[2 * v + 1] = h.x != INF32 ? h.y : INF64;
    }
    const uint64_t src_mark = mark_of(a, a.src >> a.lgK);
    uint32_t *mw = reinterpret_cast<uint32_t *>(a.mark);
    for (uint64_t i = t0; i < (uint64_t)a.W * a.mstride / 2; i += stride)
        mw[i] = i == src_mark / 4 ? phase_tag(0) << (8 * (src_mark & 3)) : 0u;
    uint32_t *c = reinterpret_cast<uint32_t *>(ctl);
    for (uint64_t i = t0; i < sizeof(ResCtl) / 4; i += stride) c[i] = 0;
}

// The selector's choice by one wavefront (features and network of selector.h, the sums in the same
// order), the weights from a copy in LDS in which lane j's inputs lie 64 apart.
__device__ __forceinline__ void learn_weights(const float *w, float *L, uint32_t tid, uint32_t bs) {
    for (uint32_t i = tid; i < kMlpParams; i += bs) {
        uint32_t to = i;  // biases and W3 stay
        if (i < kOffB1) to = i % kMlpIn * kMlpH + i / kMlpIn;
        else if (i >= kOffW2 && i < kOffB2) to = kOffW2 + (i - kOffW2) % kMlpH * kMlpH + (i - kOffW2) / kMlpH;
        L[to] = w[i];
    }
}
__device__ __forceinline__ int learn_choose(const float *L, const FeatIn &q) {
    const uint32_t j = threadIdx.x & 63, o = j < kMlpOut ? j : kMlpOut - 1;
    float x[kMlpIn];
    features_dev(q, x);
    float acc = L[kOffB1 + j];
#pragma unroll
    for (int i = 0; i < kMlpIn; ++i) acc = fmaf(L[i * kMlpH + j], x[i], acc);
    const float h1 = acc > 0.0f ? acc : 0.0f;
    acc = L[kOffB2 + j];
#pragma unroll 8
    for (int i = 0; i < kMlpH; ++i) acc = fmaf(L[kOffW2 + i * kMlpH + j], bcast(h1, i), acc);
    const float h2 = acc > 0.0f ? acc : 0.0f;
    acc = L[kOffB3 + o];
#pragma unroll 8
    for (int i = 0; i < kMlpH; ++i) acc = fmaf(L[kOffW3 + o * kMlpH + i], bcast(h2, i), acc);
    int best = 0;
    float z = bcast(acc, 0);
    for (int c = 1; c < 3; ++c) {
        const float y = bcast(acc, c);
        if (y > z) {
            z = y;
            best = c;
        }
    }
    return best;
}

// One solve by a team of a.W workgroups, this one the wg-th. Boxes, marks and distances are set up
// and visible to the team; nb counts the team's barriers. Returns the number of phases (rounds), or
// INF32 when a workgroup did not arrive in time (a.error is set).
template <int BS, int K, int IN, int OUT, bool DELTA, bool LEARN = false>
__device__ __forceinline__ uint32_t resident_run(const ResArgs &a, uint32_t wg, uint32_t &nb) {
    extern __shared__ unsigned long long dyn[];
    constexpr uint32_t kWv = BS / 64, kR = 64 / K;
    constexpr bool SIMPLE = IN == IN_SIMPLE_M || OUT == OUT_SIMPLE_M;
    __shared__ unsigned long long s_red[2 * kWv];
    __shared__ unsigned long long s_all[2 * (kResMaxW / 64)];
    __shared__ uint32_t s_wn[kWv], s_wl[kWv];  // per list: segments reserved, first reservation that failed
    __shared__ uint32_t s_pend, s_nsh, s_shlim, s_flags;
    __shared__ uint32_t s_sh[kResMaxW + 1];    // exclusive prefix of the workgroups' shared records
    __shared__ unsigned long long s_learn[8];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t li = lane & (K - 1);        // the lane's vertex in its row's group
    const uint32_t W = a.W, NS = a.mstride, n = a.n, nj = a.wslots / 64, ws0 = wave * a.wslots;
    // segments: each wavefront cuts and relaxes its own; with `share`, all go to one list whose
    // segments the workgroup's rows take in turn
    const uint32_t lw = a.share ? 0u : wave, rows = a.share ? BS / kSegEdges : 64 / kSegEdges;
    const uint32_t row0 = (a.share ? tid : lane) / kSegEdges, room = a.share ? kWv * kWaveSegs : kWaveSegs;
    Seg *seg = reinterpret_cast<Seg *>(dyn) + lw * kWaveSegs;
    unsigned long long *gk = dyn + 2 * kWv * kWaveSegs, *gd = gk + NS, *go = gd + NS;
    uint16_t *sset = reinterpret_cast<uint16_t *>(go + NS), *pend = sset + NS;
    uint16_t *rset = reinterpret_cast<uint16_t *>(gk);  // Delta-stepping: vertices the bucket removed
    uint16_t *lst = pend + NS + ws0;  // the wavefront's active slots

    for (uint32_t s = tid; s < NS; s += BS) {
        gk[s] = gd[s] = go[s] = INF64;
        sset[s] = pend[s] = 0;
    }
    if (DELTA) {
        __syncthreads();  // rset lies in gk
        for (uint32_t s = tid; s < NS; s += BS) rset[s] = 0;
    }
    if (tid == 0) {
        s_pend = s_nsh = s_flags = 0;
        s_shlim = kShareCap;
    }
    if (lane == 0) {
        s_wn[wave] = 0;
        s_wl[wave] = a.quota;
    }
    const uint64_t mall = (uint64_t)W * a.mstride;  // marks of one parity
    const uint8_t *mk = a.mark + (uint64_t)wg * a.mstride + ws0;
    gk += ws0;  // from here on the wavefront's own slots only
    gd += ws0;
    go += ws0;
    sset += ws0;
    rset += ws0;
    pend += ws0;
    auto first_vertex = [&](uint32_t s) { return ((((s * kWv + wave) << a.lgW) | wg)) * K; };
    unsigned long long *myshare = a.rec + 2ull * kShareCap * wg;
    unsigned long long minD = 0, T = OUT && !SIMPLE ? min_out64(a.vmin[a.src].y, a.wmax, a.rp, a.src) : 0ull;
    __syncthreads();

    // Cuts the row [r0, r0 + deg) of a settled vertex at distance d into segments of this
    // wavefront's list; false when they do not fit in cap.
    auto push_own = [&](uint32_t r0, uint32_t deg, unsigned long long d, uint32_t cap) {
        const uint32_t ns = ceil_div(deg, kSegEdges), p = atomicAdd(&s_wn[lw], ns);
        if (p + ns > cap) {
            atomicMin(&s_wl[lw], p);  // reservations only grow, so every later one fails too
            return false;
        }
        for (uint32_t i = 0; i < ns; ++i)
            seg[p + i] = Seg{r0 + i * kSegEdges, umin32(deg - i * kSegEdges, kSegEdges), d};
        return true;
    };
    // Reserves nr shared records; their index, or kShareCap when there is no room.
    auto reserve_shared = [&](uint32_t nr) {
        const uint32_t q = atomicAdd(&s_nsh, nr);
        if (q < kShareCap && nr <= kShareCap - q) return q;
        atomicMin(&s_shlim, q);
        return kShareCap;
    };
    auto write_shared = [&](uint32_t q, uint32_t e, uint32_t len, unsigned long long d) {
        st_agent(&myshare[2 * q], ((unsigned long long)len << 32) | e);
        st_agent(&myshare[2 * q + 1], d);
    };

    // Delta-stepping: minD is the window's lower end, hi its upper one; round kinds 0 = first
    // light round of a bucket, 1 = later light round, 2 = heavy round
    int kind = 0;
    unsigned long long hi = a.delta;
    // SIMPLE criteria: groups whose minimum of d + OUT term lies below `guess` are refreshed unasked
    unsigned long long guess = 0;
    auto in_term = [&](uint2 mm, uint2 h) { return IN != IN_SIMPLE_M ? min_in_test(mm.x) : h.x != INF32 ? h.y : INF64; };
    auto out_term = [&](uint2 mm, uint2 h, uint32_t v) {
        return OUT != OUT_SIMPLE_M ? min_out64(mm.y, a.wmax, a.rp, v) : h.x != INF32 ? h.y : INF64;
    };
    // Learned checkpoint solves: this wavefront's counts (m_reach and improving by lane), what of them
    // it has reported, and the last checkpoint's snapshot
    uint32_t l_reached = 0, l_settled = 0, l_sent_r = 0, l_sent_s = 0, l_deg = 0, l_imp = 0;
    unsigned long long l_sumf = 0, l_fprev = 0, l_sp = 0, l_min_d = 0, l_t = 0;
    float *l_w = reinterpret_cast<float *>(reinterpret_cast<char *>(dyn) + a.mlp_lds);
    auto learn_end = [&]() {  // leaves the counts in the records' place, which nobody reads any more
        const uint32_t deg = wave_sum32(l_deg), imp = wave_sum32(l_imp);  // each at most m < 2^32 in all
        if (lane == 0) {
            atomicAdd(&s_learn[3], (unsigned long long)l_reached);
            atomicAdd(&s_learn[4], (unsigned long long)l_settled);
            atomicAdd(&s_learn[5], l_sumf);
            atomicAdd(&s_learn[6], (unsigned long long)deg);
            atomicAdd(&s_learn[7], (unsigned long long)imp);
        }
        __syncthreads();
        if (tid < 5) myshare[tid] = s_learn[3 + tid];
        if (wg == 0 && tid == 0) {
            a.learn->out.min_d = minD;
            a.learn->out.t = T;
        }
    };
    if (LEARN) {
        if (tid < 8) s_learn[tid] = 0;
        if (wg == 0) learn_weights(a.mlp_w, l_w, tid, BS);
        __syncthreads();
    }
    for (uint32_t k = 0; minD != INF64; ++k) {
        const uint32_t par = k & 1;
        if (LEARN && k % 16 == 0 && k > 0) {
            // checkpoint j looks at phase 16 j + 15; its choice holds from phase 16 (j + 2) on
            if (k >= 32 && ld64(&a.learn->choice[k / 16 & 1]) != 0) {
                learn_end();
                return k;
            }
            if (wg == 0 && wave == 0) {
                FeatIn q;
                const unsigned long long r = 1 + ld64(&a.learn->sum[0]), st = ld64(&a.learn->sum[1]), sp = ld64(&a.learn->sum[2]);
                q.n = n;
                q.m = a.m;
                q.F = q.D = r - st;
                q.S = st;
                q.R = r;
                q.a = l_min_d;
                q.t = l_t;
                q.SD = q.DG = q.Ip = q.Op = 0;
                q.Fp = l_fprev;
                q.Sp = sp - l_sp;
                q.k = k;
                q.Wm = a.wm;
                q.delta_mode = 2;
                const int c = learn_choose(l_w, q);
                if (lane == 0) st_agent(&a.learn->choice[(k / 16 - 1) & 1], (unsigned long long)c);
                l_fprev = q.F;
                l_sp = sp;
            }
        }
        const uint8_t pt = (uint8_t)phase_tag(k);
        if constexpr (SIMPLE) {
            // The barrier of step 4 between refresh and certify; false when a workgroup did not arrive in
            // time. (Step 4 itself stays spelled out: as a call of this it takes 18 more registers and 1 to
            // 3 % of the time of the static criteria.)
            auto meet = [&](unsigned long long tag, unsigned long long *bar_a, unsigned long long fm, unsigned long long ft,
                            unsigned long long &pm, unsigned long long &pt2) {
                fm = wave_min_rel(fm, minD);
                if (OUT) ft = wave_min_rel(ft, minD);
                if (lane == 0) {
                    s_red[wave] = fm;
                    if (OUT) s_red[kWv + wave] = ft;
                }
                __builtin_amdgcn_s_waitcnt(0);  // this thread's stores have completed
                __syncthreads();
                if (wave == 0) {  // lanes below kWv: the minima, the next kWv: the thresholds
                    unsigned long long x = lane < (OUT ? 2 * kWv : kWv) ? s_red[lane] : INF64;
                    x = umin64(x, dpp64<kDppQuadSwap1>(x));
                    x = umin64(x, dpp64<kDppQuadSwap2>(x));
                    if (kWv >= 8) x = umin64(x, dpp64<kDppHalfMirror>(x));
                    if (kWv >= 16) x = umin64(x, dpp64<kDppMirror>(x));
                    if (lane == 0 || (OUT && lane == kWv))
                        st_agent(&bar_a[wg * kSlotStride + (lane ? 1 : 0)], tag | umin64(x, kVal));
                }
                pm = pt2 = kVal;
                if (tid < W) {
                    const unsigned long long *w = &bar_a[tid * kSlotStride];
                    uint32_t spins = 0;
                    for (;;) {
                        pm = ld64(w);
                        if (OUT) pt2 = ld64(w + 1);
                        if ((pm & kTag) == tag && (!OUT || (pt2 & kTag) == tag)) break;
                        if (++spins >= a.polls) {
                            atomicOr(&s_flags, 1u);
                            break;
                        }
                    }
                    pm &= kVal;
                    if (OUT) pt2 &= kVal;
                }
                if (wave * 64 < W) {
                    pm = wave_min_rel(pm == kVal ? INF64 : pm, minD);
                    if (OUT) pt2 = wave_min_rel(pt2 == kVal ? INF64 : pt2, minD);
                    if (lane == 0) {
                        s_all[wave] = pm;
                        s_all[kResMaxW / 64 + wave] = pt2;
                    }
                }
                __syncthreads();
                if (s_flags & 1u) {  // block-uniform
                    if (tid == 0) atomicOr(a.error, 1u);
                    return false;
                }
                pm = s_all[0];
                pt2 = s_all[kResMaxW / 64];
                for (uint32_t i = 1; i * 64 < W; ++i) {
                    pm = umin64(pm, s_all[i]);
                    pt2 = umin64(pt2, s_all[kResMaxW / 64 + i]);
                }
                pm = readlane64(pm, 0);
                if (OUT) pt2 = readlane64(pt2, 0);
                return true;
            };
            uint32_t na = 0;
            auto list = [&](uint32_t j, bool act) {
                const unsigned long long mask = __ballot(act);
                if (act) lst[na + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull))] = (uint16_t)(j * 64 + lane);
                na += (uint32_t)__popcll(mask);
            };
            {
                uint8_t m[kMaxJ];
#pragma unroll
                for (uint32_t j = 0; j < kMaxJ; ++j) {
                    m[j] = 0;
                    if (j < nj) m[j] = __hip_atomic_load(mk + j * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (uint32_t j = 0; j < kMaxJ; ++j) {
                    if (j >= nj) break;  // block-uniform
                    const unsigned long long o = OUT == OUT_SIMPLE_M ? go[j * 64 + lane] : INF64;
                    list(j, m[j] == pt || (o != INF64 && o <= guess));
                }
            }
            // Brings the listed groups' minima up to date. An OUT head is looked at only where the sum it
            // was last seen with is at most `limit`: it only grows, so larger ones stay larger.
            auto refresh = [&](unsigned long long limit) {
                struct Vert {
                    uint32_t s, v, cur, end;
                    unsigned long long d;
                    uint2 mm, hi, ho;
                };
                auto load = [&](uint32_t i0) {
                    Vert c{INF32, 0u, 0u, 0u, INF64, make_uint2(INF32, INF32), make_uint2(INF32, INF32), make_uint2(INF32, INF32)};
                    const uint32_t i = i0 + lane / K;
                    if (i < na) {
                        c.s = lst[i];
                        c.v = first_vertex(c.s) + li;
                        if (c.v < n) {
                            c.d = ld64(&a.box[2ull * c.v]);
                            if (IN == IN_SIMPLE_M) {
                                c.hi = a.in_head[c.v];
                                c.cur = a.in_cur[c.v];
                                c.end = a.ip[c.v + 1];
                            }
                            if (OUT == OUT_SIMPLE_M) c.ho = a.out_head[c.v];
                            if (IN == IN_STATIC_M || OUT == OUT_STATIC_M) c.mm = a.vmin[c.v];
                        }
                    }
                    return c;
                };
                struct Next {
                    uint2 e[2];
                };
                auto next_edges = [&](const uint2 *row, uint32_t cur, uint32_t end) {
                    Next x;
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        x.e[q] = make_uint2(INF32, INF32);
                        if (cur + q < end) x.e[q] = row[cur + q];
                    }
                    return x;
                };
                // h: the first edge at or after row[cur] whose other end has not settled; x holds the next two.
                // Two at a time, read before it is known that the head settled: of the vertices looked at
                // few move and most of these by one (four at a time 3 to 4 % slower, none ahead 2 to 5 %)
                auto advance = [&](uint2 &h, uint32_t &cur, Next x, const uint2 *row, uint32_t end) {
                    for (;;) {
                        unsigned long long d[2];
#pragma unroll
                        for (int q = 0; q < 2; ++q) d[q] = x.e[q].x != INF32 ? ld64(&a.box[2ull * x.e[q].x]) : INF64;
                        h = make_uint2(INF32, INF32);
                        uint32_t step = 2;
#pragma unroll
                        for (int q = 1; q >= 0; --q)
                            if (!dist_settled(d[q])) {  // an edge, or the end of the row
                                h = x.e[q];
                                step = q;
                            }
                        cur += step;
                        if (step < 2) return;
                        x = next_edges(row, cur, end);
                    }
                };
                wave_fence();
                Vert nxt = load(0);
                for (uint32_t i0 = 0; i0 < na; i0 += kR) {
                    Vert c = nxt;
                    if (i0 + kR < na) nxt = load(i0 + kR);
                    const bool q = !(c.d >> 63);  // queued: neither infinite nor settled
                    const bool qi = IN == IN_SIMPLE_M && q && c.hi.x != INF32;
                    const bool qo = OUT == OUT_SIMPLE_M && q && c.ho.x != INF32 && sadd64(c.d, c.ho.y) <= limit;
                    unsigned long long xi = INF64, xo = INF64;
                    uint32_t ocur = 0, oend = 0;
                    if (qo) {
                        xo = ld64(&a.box[2ull * c.ho.x]);
                        ocur = a.out_cur[c.v] + 1;
                        oend = a.rp[c.v + 1];
                    }
                    if (qi) {
                        xi = ld64(&a.box[2ull * c.hi.x]);
                        const Next x = next_edges(a.in_edges, ++c.cur, c.end);
                        if (dist_settled(xi)) {
                            advance(c.hi, c.cur, x, a.in_edges, c.end);
                            a.in_cur[c.v] = c.cur;
                            a.in_head[c.v] = c.hi;
                            st_agent(&a.box[2ull * c.v + 1], c.hi.x != INF32 ? (unsigned long long)c.hi.y : INF64);
                        }
                    }
                    if (dist_settled(xo)) {
                        advance(c.ho, ocur, next_edges(a.edges, ocur, oend), a.edges, oend);
                        a.out_cur[c.v] = ocur;
                        a.out_head[c.v] = c.ho;
                    }
                    if (q) a.dist[c.v] = c.d;
                    const unsigned long long mi = in_term(c.mm, c.hi), mo = out_term(c.mm, c.ho, c.v);
                    // keys below the last minD pass any test: cut off there, where the minima are based
                    unsigned long long key = c.d > mi ? c.d - mi : 0ull;
                    if (key < minD) key = minD;
                    const unsigned long long rk = IN != IN_NONE ? row_min_rel<K>(q ? key : INF64, minD) : INF64;
                    const unsigned long long rd = row_min_rel<K>(q ? c.d : INF64, minD);
                    const unsigned long long ro = OUT ? row_min_rel<K>(q ? sadd64(c.d, mo) : INF64, minD) : INF64;
                    if (c.s != INF32 && li == 0) {
                        if (IN != IN_NONE) gk[c.s] = rk;
                        gd[c.s] = rd;
                        if (OUT) go[c.s] = ro;
                    }
                }
                wave_fence();
            };
            unsigned long long pm, pt2;
            for (;;) {
                refresh(guess);
                unsigned long long fm = INF64, ft = INF64;
#pragma unroll
                for (uint32_t j = 0; j < kMaxJ; ++j)
                    if (j < nj) {
                        fm = umin64(fm, gd[j * 64 + lane]);
                        if (OUT) ft = umin64(ft, go[j * 64 + lane]);
                    }
                if (!meet(bar_tag(nb), a.bar + bar_words(nb, W), fm, ft, pm, pt2)) return INF32;
                ++nb;
                // sums up to the guess are exact, larger ones lower bounds
                if (OUT != OUT_SIMPLE_M || pt2 == INF64 || pt2 <= guess) break;
                const unsigned long long seen = guess;
                guess = sadd64(pt2, 4 * (pt2 - pm));
                na = 0;
#pragma unroll
                for (uint32_t j = 0; j < kMaxJ; ++j)
                    if (j < nj) {
                        const unsigned long long o = go[j * 64 + lane];
                        list(j, o > seen && o <= guess && o != INF64);
                    }
            }
            if (pm == INF64) return k;  // nothing is queued
            if (k > a.max_phases) {
                if (tid == 0) atomicOr(a.error, 2u);
                return INF32;
            }
            minD = pm;
            T = pt2;
            guess = sadd64(T, 4 * (T - minD));
        }
        const unsigned long long tag = bar_tag(nb);
        unsigned long long *bar_a = a.bar + bar_words(nb, W), *bar_b = a.bar + count_words(W);
        ++nb;
        // 1. the wavefront's active groups
        uint32_t na = 0;  // wavefront-uniform
        {
            uint8_t m[kMaxJ];
#pragma unroll
            for (uint32_t j = 0; j < kMaxJ; ++j) {
                m[j] = 0;
                if (!SIMPLE && j < nj) m[j] = __hip_atomic_load(mk + par * mall + j * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (uint32_t j = 0; j < kMaxJ; ++j) {
                if (j >= nj) break;  // block-uniform
                const uint32_t s = j * 64 + lane;
                const unsigned long long d = gd[s];
                const bool act = (!SIMPLE && m[j] == pt) || (IN != IN_NONE && gk[s] <= minD) || (OUT && d != INF64 && d <= T) ||
                                 (DELTA && (kind == 0 ? d < hi : kind == 2 && rset[s] != 0));
                const unsigned long long mask = __ballot(act);
                if (act) lst[na + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull))] = (uint16_t)s;
                na += (uint32_t)__popcll(mask);
            }
        }
        wave_fence();
        // 2. identify: kR groups per step, the next step's loads issued before this one's work
        struct Cand {
            uint32_t s, v, r0, r1;
            unsigned long long d, x;
            uint2 mm, hi, ho;  // static minima, heads
        };
        auto load = [&](uint32_t i0) {
            Cand c{INF32, 0u, 0u, 0u, INF64, INF64, make_uint2(INF32, INF32), make_uint2(INF32, INF32), make_uint2(INF32, INF32)};
            const uint32_t i = i0 + lane / K;
            if (i < na) {
                c.s = lst[i];
                c.v = first_vertex(c.s) + li;
                if (c.v < n) {
                    c.d = a.dist[c.v];
                    if (!SIMPLE) c.x = ld64(&a.box[2ull * c.v + par]);
                    if (IN != IN_SIMPLE_M || OUT == OUT_STATIC_M) c.mm = a.vmin[c.v];
                    if (IN == IN_SIMPLE_M) c.hi = a.in_head[c.v];
                    if (OUT == OUT_SIMPLE_M) c.ho = a.out_head[c.v];
                    c.r0 = a.rp[c.v];
                    c.r1 = a.rp[c.v + 1];
                }
            }
            return c;
        };
        bool waiting = false;  // wavefront-uniform: some settled rows found no room
        uint32_t l_now = 0;    // settled in this phase
        Cand nxt = load(0);
        for (uint32_t i0 = 0; i0 < na; i0 += kR) {
            Cand c = nxt;
            if (i0 + kR < na) nxt = load(i0 + kR);
            const bool lowered = c.x < c.d;  // by the last phase's relaxes
            if (LEARN) {
                const uint32_t r = (uint32_t)__popcll(__ballot(lowered && c.d == INF64));
                l_reached += r;
                l_sumf -= (unsigned long long)k * r;
            }
            if (lowered) {
                c.d = c.x;
                a.dist[c.v] = c.x;
            }
            const bool removed = DELTA && c.s != INF32 && ((uint32_t)rset[c.s] >> li & 1u);
            const bool q = c.d != INF64 && !((uint32_t)sset[c.s] >> li & 1u);  // d is INF64 without a group
            const unsigned long long mi = in_term(c.mm, c.hi);
            const unsigned long long key = IN == IN_DIJK ? c.d : c.d > mi ? c.d - mi : 0ull;  // d - minIn
            bool ok = false;
            if (IN != IN_NONE) ok = key <= minD;  // eq. crit:instatic
            if (OUT) ok = ok || c.d <= T;         // eq. crit:outstatic
            if (DELTA) ok = kind == 2 ? removed : c.d < hi && (kind == 0 || lowered);
            ok = ok && q;
            if (SIMPLE && ok) st_agent(&a.box[2ull * c.v], c.d | kSettledBit);
            const uint32_t deg = c.r1 - c.r0;
            bool wait = false;
            const unsigned long long okm = __ballot(ok);
            if (LEARN) {
                const uint32_t r = (uint32_t)__popcll(okm);
                l_settled += r;
                l_now += r;
                l_sumf += (k + 1ull) * r;
                if (ok) {
                    l_deg += deg;
                    a.sp[c.v] = k + 1;
                }
            }
            if (okm) {
                if (ok && deg > 0 && deg <= kHubEdges) {
                    if (!push_own(c.r0, deg, c.d, a.quota)) {
                        const uint32_t nr = ceil_div(deg, kShareEdges), qi = a.share ? reserve_shared(nr) : kShareCap;
                        wait = qi == kShareCap;
                        if (!wait)
                            for (uint32_t i = 0; i < nr; ++i)
                                write_shared(qi + i, c.r0 + i * kShareEdges,
                                             umin32(deg - i * kShareEdges, kShareEdges), c.d);
                    }
                }
                for (unsigned long long hm = __ballot(ok && deg > kHubEdges); hm; hm &= hm - 1) {
                    const int l = __ffsll((long long)hm) - 1;
                    const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)c.r0, l);
                    const uint32_t dg = (uint32_t)__builtin_amdgcn_readlane((int)deg, l);
                    const unsigned long long hd = readlane64(c.d, l);
                    uint32_t len = kShareEdges;
                    while (ceil_div(dg, len) > kShareCap / 2) len *= 2;
                    const uint32_t nr = ceil_div(dg, len);
                    uint32_t qi = 0;
                    if (lane == 0) qi = a.share ? reserve_shared(nr) : kShareCap;
                    qi = (uint32_t)__builtin_amdgcn_readlane((int)qi, 0);
                    if (qi == kShareCap) wait = wait || (int)lane == l;
                    else
                        for (uint32_t i = lane; i < nr; i += 64) write_shared(qi + i, e + i * len, umin32(dg - i * len, len), hd);
                }
            }
            const bool keep = q && !ok && !removed;
            const unsigned long long rk = IN != IN_NONE ? row_min_rel<K>(keep ? key : INF64, minD) : INF64;
            const unsigned long long rd = row_min_rel<K>(keep ? c.d : INF64, minD);
            const unsigned long long ro =
                OUT ? row_min_rel<K>(keep ? sadd64(c.d, out_term(c.mm, c.ho, c.v)) : INF64, minD) : INF64;
            const unsigned long long wm = __ballot(wait);
            waiting = waiting || wm != 0;
            if (c.s != INF32 && li == 0) {
                const uint32_t sh = lane & ~(K - 1u), low = (1u << K) - 1u;
                if (IN != IN_NONE) gk[c.s] = rk;
                gd[c.s] = rd;
                if (OUT) go[c.s] = ro;
                if (okm >> sh & low) {
                    if (!DELTA || kind == 2) sset[c.s] |= (uint16_t)(okm >> sh & low);
                    if (DELTA) rset[c.s] = kind == 2 ? 0 : (uint16_t)(rset[c.s] | (okm >> sh & low));
                }
                if (wm >> sh & low) pend[c.s] = (uint16_t)(wm >> sh & low);
            }
        }
        if (LEARN && k % 16 == 15) {
            if (lane == 0) {
                atomicAdd(&s_learn[0], (unsigned long long)(l_reached - l_sent_r));
                atomicAdd(&s_learn[1], (unsigned long long)(l_settled - l_now - l_sent_s));
                atomicAdd(&s_learn[2], (unsigned long long)l_now);
            }
            l_sent_r = l_reached;
            l_sent_s = l_settled - l_now;
            l_min_d = minD;
            l_t = T;
        }
        if (a.share) {
            if (waiting && lane == 0) s_pend = 1;
            __builtin_amdgcn_s_waitcnt(0);  // this wavefront's records are written
            __syncthreads();
            if (tid == 0 && W > 1) st_agent(&bar_b[wg * kSlotStride], count_word(nb, umin32(s_nsh, s_shlim)));
        }
        wave_fence();
        uint32_t nseg = umin32(s_wn[lw], s_wl[lw]);
        // 3. relax. A candidate below both of its target's boxes passes. Together they hold the target's
        // distance at phase start (and perhaps lower candidates of this phase), so none passes towards
        // a settled target. Folding one that another candidate of this phase undercuts changes no
        // minimum, since the lower one is folded too, so the atomic returns nothing.
        unsigned long long fm = INF64, ft = INF64;
        const uint8_t nt = (uint8_t)phase_tag(k + 1);
        auto apply = [&](uint2 ed, uint32_t em, unsigned long long cur, unsigned long long d) {
            const unsigned long long cand = d + ed.y;
            if constexpr (SIMPLE) {  // em: the target's IN term, which the settling of this edge's source may raise
                if (dist_settled(cur)) return;
                if (cand < cur)
                    (void)__hip_atomic_fetch_min(&a.box[2ull * ed.x], cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (cand < cur || (IN == IN_SIMPLE_M && ed.y == em)) st_agent(a.mark + mark_of(a, ed.x / K), nt);
                return;
            }
            if (cand >= cur) return;
            const unsigned long long old =
                __hip_atomic_fetch_min(&a.box[2ull * ed.x + (par ^ 1)], cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (LEARN) l_imp += cand < old;
            st_agent(a.mark + (par ^ 1) * mall + mark_of(a, ed.x / K), nt);
            if (!DELTA || kind == 2 || cand < hi) fm = umin64(fm, cand);
            if (OUT) ft = umin64(ft, sadd64(cand, min_out64(em, a.wmax, a.rp, ed.x)));
        };
        constexpr unsigned long long none = SIMPLE ? kSettledBit : 0ull;  // the target word of a lane without an edge
        // Delta-stepping: light rounds take edges below the width, the heavy round the others
        auto takes = [&](uint32_t w) { return !DELTA || (w < a.delta) == (kind != 2); };
        auto target = [&](uint32_t v) {
            if (SIMPLE) return ld64(&a.box[2ull * v]);
            return umin64(ld64(&a.box[2ull * v]), ld64(&a.box[2ull * v + 1]));
        };
        auto extra = [&](uint64_t e, uint32_t v) {  // of an edge: what apply takes as em
            if (IN == IN_SIMPLE_M) return (uint32_t)ld64(&a.box[2ull * v + 1]);
            return OUT && !SIMPLE ? a.emin[e] : INF32;
        };
        // relaxes edges [e, e + len) at distance d by the wavefront
        auto relax_range = [&](uint32_t e, uint32_t len, unsigned long long d) {
            for (uint64_t j0 = lane; j0 < len; j0 += 256) {
                uint2 he[4];
                uint32_t hm[4];
                unsigned long long hc[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    he[j] = make_uint2(0u, 0u);
                    hm[j] = INF32;
                    if (j0 + j * 64 < len) {
                        he[j] = a.edges[e + j0 + j * 64];
                        if (!SIMPLE) hm[j] = extra(e + j0 + j * 64, 0u);
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    hc[j] = none;
                    if (j0 + j * 64 < len && takes(he[j].y)) {
                        hc[j] = target(he[j].x);
                        if (SIMPLE) hm[j] = extra(0, he[j].x);
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) apply(he[j], hm[j], hc[j], d);
            }
        };
        uint2 ed = make_uint2(0u, 0u);
        uint32_t em = INF32;
        unsigned long long cur = none, sd = 0;
        auto fetch = [&](uint32_t i) {  // lane l of a row of 16: edge l of segment i
            cur = none;
            if (i < nseg) {
                const Seg sg = seg[i];
                const uint32_t l = lane & (kSegEdges - 1);
                if (l < sg.len) {
                    ed = a.edges[sg.e + l];
                    em = extra(sg.e + l, ed.x);
                    sd = sg.d;
                    if (takes(ed.y)) cur = target(ed.x);
                }
            }
        };
        auto relax_own = [&]() {  // the first step's edges are fetched
            for (uint32_t i = row0; __ballot(i < nseg); i += rows) {
                const uint2 ped = ed;
                const uint32_t pem = em;
                const unsigned long long pcur = cur, psd = sd;
                fetch(i + rows);  // before this step's atomics, so that its loads do not queue behind them
                apply(ped, pem, pcur, psd);
            }
        };
        fetch(row0);
        // the workgroup's minima over what it keeps
#pragma unroll
        for (uint32_t j = 0; j < kMaxJ; ++j)
            if (!SIMPLE && j < nj && (!DELTA || kind == 2)) {
                fm = umin64(fm, gd[j * 64 + lane]);
                if (OUT) ft = umin64(ft, go[j * 64 + lane]);
            }
        relax_own();
        // Rows that found no room, as many as fit: segments of this wavefront's pending vertices
        // (hubs are relaxed at once). True if some are left.
        auto refill = [&]() {
            bool full = false, left = false;
            for (uint32_t j = 0; j < nj; ++j) {
                const uint32_t s = j * 64 + lane;
                uint32_t p = pend[s];
                while (!full && __ballot(p != 0)) {
                    uint32_t r0 = 0, deg = 0;
                    unsigned long long d = 0;
                    if (p) {
                        const uint32_t v = first_vertex(s) + __ffs(p) - 1;
                        r0 = a.rp[v];
                        deg = a.rp[v + 1] - r0;
                        d = a.dist[v];
                    }
                    const bool hub = deg > kHubEdges;
                    const bool took = hub || (p && push_own(r0, deg, d, room));
                    for (unsigned long long hm = __ballot(hub); hm; hm &= hm - 1) {
                        const int l = __ffsll((long long)hm) - 1;
                        relax_range((uint32_t)__builtin_amdgcn_readlane((int)r0, l),
                                    (uint32_t)__builtin_amdgcn_readlane((int)deg, l), readlane64(d, l));
                    }
                    full = __ballot(p && !took) != 0;
                    if (took) p &= p - 1;
                }
                pend[s] = (uint16_t)p;
                left = left || __ballot(p != 0) != 0;
            }
            return left;
        };
        while (!a.share && waiting) {  // wavefront-uniform
            wave_fence();
            if (lane == 0) {
                s_wn[wave] = 0;
                s_wl[wave] = room;
            }
            wave_fence();
            waiting = refill();
            wave_fence();
            nseg = umin32(s_wn[wave], s_wl[wave]);
            fetch(row0);
            relax_own();
        }
        if (a.share) {
            if (W == 1) {
                if (tid == 0) {
                    s_sh[0] = umin32(s_nsh, s_shlim);
                    if (s_sh[0]) s_flags |= 2u;
                }
            } else if (tid < W) {
                uint32_t spins = 0;
                unsigned long long v;
                while (!count_is_for(v = ld64(&bar_b[tid * kSlotStride]), nb) && ++spins < a.polls) {}
                s_sh[tid] = (uint32_t)v;
                if (!count_is_for(v, nb)) atomicOr(&s_flags, 1u);
                else if ((uint32_t)v) atomicOr(&s_flags, 2u);
            }
            __syncthreads();
            uint32_t pending = s_pend;
            if (s_flags == 2u) {  // block-uniform
                if (wave == 0) {  // counts to an exclusive prefix, four per lane
                    uint32_t c[4], sum = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        c[j] = 4 * lane + j < W ? s_sh[4 * lane + j] : 0u;
                        sum += c[j];
                    }
                    const uint32_t incl = wave_incl_scan(sum);
                    uint32_t o = incl - sum;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (4 * lane + j < W) s_sh[4 * lane + j] = o;
                        o += c[j];
                    }
                    if (lane == 63) s_sh[W] = incl;
                }
                __syncthreads();
                const uint32_t shared = s_sh[W];
                // one record per wavefront, spread over the workgroups first
                for (uint32_t r = wg + W * wave; r < shared; r += W * kWv) {
                    uint32_t lo = 0;  // last workgroup whose first record is <= r
                    for (uint32_t st = W / 2; st > 0; st >>= 1)
                        if (s_sh[lo + st] <= r) lo += st;
                    const unsigned long long *rec = a.rec + 2ull * (kShareCap * lo + (r - s_sh[lo]));
                    const unsigned long long x = ld64(rec), d = ld64(rec + 1);
                    relax_range((uint32_t)x, (uint32_t)(x >> 32), d);
                }
            }
            while (pending) {  // block-uniform
                __syncthreads();
                if (tid == 0) {
                    s_pend = s_wn[0] = 0;
                    s_wl[0] = room;
                }
                __syncthreads();
                if (refill() && lane == 0) s_pend = 1;
                __syncthreads();
                pending = s_pend;
                nseg = umin32(s_wn[0], s_wl[0]);
                fetch(row0);
                relax_own();
            }
        }
        // 4. combine: publish this workgroup's minima and read everybody's
        fm = wave_min_rel(fm, minD);
        if (OUT) ft = wave_min_rel(ft, minD);
        if (lane == 0) {
            s_red[wave] = fm;
            if (OUT) s_red[kWv + wave] = ft;
        }
        __builtin_amdgcn_s_waitcnt(0);  // this thread's atomics and marks have completed
        __syncthreads();
        if (lane == 0) {
            s_wn[wave] = 0;
            s_wl[wave] = a.quota;
        }
        if (tid == 0) {
            s_pend = s_nsh = 0;
            atomicAnd(&s_flags, 1u);  // another wavefront may be giving up
            s_shlim = kShareCap;
        }
        if (LEARN && k % 16 == 15 && wave == 0) {
            if (lane < 3) {
                atomicAdd(&a.learn->sum[lane], s_learn[lane]);
                s_learn[lane] = 0;
            }
            __builtin_amdgcn_s_waitcnt(0);
        }
        if (wave == 0) {  // lanes below kWv: the minima, the next kWv: the thresholds
            unsigned long long x = lane < (OUT ? 2 * kWv : kWv) ? s_red[lane] : INF64;
            x = umin64(x, dpp64<kDppQuadSwap1>(x));
            x = umin64(x, dpp64<kDppQuadSwap2>(x));
            if (kWv >= 8) x = umin64(x, dpp64<kDppHalfMirror>(x));
            if (kWv >= 16) x = umin64(x, dpp64<kDppMirror>(x));
            if (lane == 0 || (OUT && lane == kWv)) {
                if (W > 1) st_agent(&bar_a[wg * kSlotStride + (lane ? 1 : 0)], tag | umin64(x, kVal));
                else s_all[lane ? kResMaxW / 64 : 0] = x;  // a workgroup alone waits for no words
            }
        }
        unsigned long long pm = kVal, pt2 = kVal;
        if (W > 1 && tid < W) {
            const unsigned long long *w = &bar_a[tid * kSlotStride];
            uint32_t spins = 0;
            for (;;) {
                pm = ld64(w);
                if (OUT) pt2 = ld64(w + 1);
                if ((pm & kTag) == tag && (!OUT || (pt2 & kTag) == tag)) break;
                if (++spins >= a.polls) {
                    atomicOr(&s_flags, 1u);
                    break;
                }
            }
            pm &= kVal;
            if (OUT) pt2 &= kVal;
        }
        if (W > 1 && wave * 64 < W) {
            pm = wave_min_rel(pm == kVal ? INF64 : pm, minD);
            if (OUT) pt2 = wave_min_rel(pt2 == kVal ? INF64 : pt2, minD);
            if (lane == 0) {
                s_all[wave] = pm;
                s_all[kResMaxW / 64 + wave] = pt2;
            }
        }
        __syncthreads();
        if (s_flags & 1u) {  // block-uniform
            if (tid == 0) atomicOr(a.error, 1u);
            return INF32;
        }
        pm = s_all[0];
        pt2 = s_all[kResMaxW / 64];
        for (uint32_t i = 1; i * 64 < W; ++i) {
            pm = umin64(pm, s_all[i]);
            pt2 = umin64(pt2, s_all[kResMaxW / 64 + i]);
        }
        pm = readlane64(pm, 0);
        if (SIMPLE) continue;  // the next phase's refresh finds minD and T
        if (!DELTA) {
            minD = pm;
            if (OUT) T = readlane64(pt2, 0);
        } else if (kind != 2) {
            kind = pm != INF64 ? 1 : 2;
        } else {
            kind = 0;
            minD = pm != INF64 ? pm / a.delta * a.delta : INF64;
            hi = sadd64(minD, a.delta);
        }
        if (k > a.max_phases) {
            if (tid == 0) atomicOr(a.error, 2u);
            return INF32;
        }
        if (minD == INF64) {
            if (LEARN) learn_end();
            return k + 1;
        }
    }
    return 0;  // not reached: the first phase settles the source
}

template <int BS, int K, int IN, int OUT, bool DELTA = false, bool LEARN = false>
__global__ __launch_bounds__(BS) void k_resident(ResArgs a, ResCtl *ctl, uint32_t one_xcd) {
    __shared__ uint32_t s_wg;
    // the workgroup's rank in the team
    uint32_t wg = blockIdx.x;
    if (one_xcd) {  // the others leave: an L2 of its own serves the whole team
        // the first XCD on which W workgroups have arrived is the team's; the launch holds 8 W
        // workgroups, so one of the eight gets there whatever their placement
        if (threadIdx.x == 0) {
            const uint32_t x = __builtin_amdgcn_s_getreg((31 << 11) | 20) & 0xfu;  // HW_REG_XCC_ID
            const uint32_t r = atomicAdd(&ctl->rank[x * 32], 1u);
            if (r == a.W - 1) atomicCAS(&ctl->team, 0u, x + 1);
            uint32_t t = 0, spins = 0;
            while (!(t = __hip_atomic_load(&ctl->team, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) && ++spins < a.polls)
                __builtin_amdgcn_s_sleep(1);
            if (!t) atomicOr(a.error, 1u);
            s_wg = t == x + 1 && r < a.W ? r : INF32;
        }
        __syncthreads();
        wg = s_wg;
        if (wg == INF32) return;
    }
    uint32_t nb = 0;
    const uint32_t phases = resident_run<BS, K, IN, OUT, DELTA, LEARN>(a, wg, nb);
    if (wg == 0 && threadIdx.x == 0 && phases != INF32) st_agent(&ctl->phases, phases);
}

// After a learned checkpoint solve's static stage: sums the workgroups' counts (block 0) and counts
// the relaxations towards targets not settled by then, from the settle phases. Each thread takes
// kCountEdges consecutive edges, whatever the rows' lengths. The static stage itself sees no settled
// flags. 16.8 M edges: 246 us (371 with the edges loaded one after the other), most of it the settle
// phases of random targets.
constexpr uint32_t kCountEdges = 16;
__global__ __launch_bounds__(256) void k_learn_counts(ResArgs a) {
    const uint32_t lane = threadIdx.x & 63;
    ResLearned &o = a.learn->out;
    if (blockIdx.x == 0) {
        unsigned long long x[5];
        for (int i = 0; i < 5; ++i) {
            x[i] = threadIdx.x < a.W ? a.rec[2ull * kShareCap * threadIdx.x + i] : 0ull;
            x[i] = wave_sum64(x[i]);
        }
        if (lane == 0) {
            atomicAdd(&o.reached, x[0]);
            atomicAdd(&o.settled, x[1]);
            atomicAdd(&o.sum_f, x[2]);
            atomicAdd(&o.m_reach, x[3]);
            atomicAdd(&o.improving, x[4]);
        }
    }
    uint32_t count = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i * kCountEdges < a.m; i += (uint64_t)gridDim.x * 256) {
        const uint64_t e0 = i * kCountEdges;
        const uint32_t len = a.m - e0 < kCountEdges ? (uint32_t)(a.m - e0) : kCountEdges;
        uint32_t to[kCountEdges], sv[kCountEdges];
#pragma unroll
        for (uint32_t q = 0; q < kCountEdges; ++q) to[q] = q < len ? a.edges[e0 + q].x : a.src;
        uint32_t u = 0, hi = a.n;  // rp[u] <= e0 < rp[hi]
        while (hi - u > 1) {
            const uint32_t mid = u + (hi - u) / 2;
            if (a.rp[mid] <= e0) u = mid;
            else hi = mid;
        }
#pragma unroll
        for (uint32_t q = 0; q < kCountEdges; ++q) sv[q] = a.sp[to[q]];  // the source settled first: past the end counts nothing
        uint64_t end = a.rp[u + 1];
        uint32_t su = a.sp[u];
#pragma unroll
        for (uint32_t q = 0; q < kCountEdges; ++q) {
            while (q < len && e0 + q >= end) {
                end = a.rp[++u + 1];
                su = a.sp[u];
            }
            count += su != 0 && (sv[q] == 0 || sv[q] > su);
        }
    }
    count = wave_sum32(count);
    if (lane == 0 && count) atomicAdd(&o.relax_edges, (unsigned long long)count);
}

// The state of a learned checkpoint solve after its static stage, as the phase kernels keep it; adds
// the vertices that the stage's last phase reached, which no owner has seen, to ctl->reached.
__global__ __launch_bounds__(256) void k_learn_state(ResArgs a, uint8_t *st, uint2 *in_head, uint2 *out_head, Ctl *ctl) {
    __shared__ uint32_t s_new;
    const uint2 none = make_uint2(INF32, INF32);
    uint32_t fresh = 0;
    if (threadIdx.x == 0) s_new = 0;
    __syncthreads();
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n; v += gridDim.x * blockDim.x) {
        const unsigned long long was = a.dist[v], d = umin64(was, umin64(a.box[2ull * v], a.box[2ull * v + 1]));
        fresh += was == INF64 && d != INF64;
        const bool settled = a.sp[v] != 0;
        a.dist[v] = settled ? d | kSettledBit : d;
        st[v] = settled ? ST_S : d != INF64 ? ST_F : ST_U;
        const uint32_t o = a.rp[v], i = a.ip[v];
        a.out_cur[v] = o;
        a.in_cur[v] = i;
        out_head[v] = o < a.rp[v + 1] ? a.edges[o] : none;
        in_head[v] = i < a.ip[v + 1] ? a.in_edges[i] : none;
    }
    if (fresh) atomicAdd(&s_new, fresh);
    __syncthreads();
    if (threadIdx.x == 0 && s_new) atomicAdd(&ctl->reached.v[blockIdx.x % kShards * kPad], (unsigned long long)s_new);
}

typedef void (*rfn)(ResArgs, ResCtl *, uint32_t);

template <int BS, int K>
static rfn pick_res_bs(int in, bool out) {
    if (in == IN_DIJK) return out ? k_resident<BS, K, IN_DIJK, true> : k_resident<BS, K, IN_DIJK, false>;
    if (in == IN_STATIC_M) return out ? k_resident<BS, K, IN_STATIC_M, true> : k_resident<BS, K, IN_STATIC_M, false>;
    return k_resident<BS, K, IN_NONE, true>;
}

template <int BS, int K>
static rfn pick_res_simple(int in, int out) {
    if (in == IN_NONE) return k_resident<BS, K, IN_NONE, OUT_SIMPLE_M>;
    if (in == IN_STATIC_M) return k_resident<BS, K, IN_STATIC_M, OUT_SIMPLE_M>;
    if (out == OUT_NONE) return k_resident<BS, K, IN_SIMPLE_M, OUT_NONE>;
    return out == OUT_STATIC_M ? k_resident<BS, K, IN_SIMPLE_M, OUT_STATIC_M> : k_resident<BS, K, IN_SIMPLE_M, OUT_SIMPLE_M>;
}

static rfn pick_res(int bs, int lgK, int in, int out, bool delta) {
    if (in == IN_SIMPLE_M || out == OUT_SIMPLE_M) {
        if (bs == 512) return lgK == 3 ? pick_res_simple<512, 8>(in, out) : pick_res_simple<512, 16>(in, out);
        return lgK == 3 ? pick_res_simple<1024, 8>(in, out) : pick_res_simple<1024, 16>(in, out);
    }
    if (delta) {
        if (bs == 512) return lgK == 3 ? k_resident<512, 8, IN_NONE, false, true> : k_resident<512, 16, IN_NONE, false, true>;
        return lgK == 3 ? k_resident<1024, 8, IN_NONE, false, true> : k_resident<1024, 16, IN_NONE, false, true>;
    }
    if (bs == 512) return lgK == 3 ? pick_res_bs<512, 8>(in, out) : pick_res_bs<512, 16>(in, out);
    return lgK == 3 ? pick_res_bs<1024, 8>(in, out) : pick_res_bs<1024, 16>(in, out);
}
// Shape by the number of edges, measured on MI355X (us per phase; random, R-MAT and grid graphs):
//   below 2^20 edges one XCD: its workgroups share an L2, so barriers and marks stay in it (grid of
//   249 k vertices: 4.4 on 32 workgroups of one XCD, 4.8 on 128 of all; R-MAT 16: 8.0 against 8.3);
//   512 threads while phases are so small that a wavefront's instructions count (below 2^18 edges).
//   Up to 2^23 edges 128 workgroups (random, 1 M vertices of degree 4: 6.3 against 6.7 on 256 and 7.1
//   on 64; grid of 1 M vertices: 5.0, 5.8 and 5.0), then one on every CU (random, 1 M vertices of
//   degree 16: 7.4 against 8.5 on 64).
// Groups of 8 vertices move half the bytes of groups of 16, which only graphs of more than 2^23
// vertices need to fit their slots into LDS. Where the slots still do not fit, the next shape is taken.
ResShape resident_shape(const sssp_graph *g) {
    struct Shape { uint64_t max_m; uint32_t W; int bs; uint32_t one_xcd, lgK; };
    static const Shape shapes[] = {{1ull << 18, 32, 512, 1, 3},   {1ull << 20, 32, 1024, 1, 3},
                                   {1ull << 23, 128, 1024, 0, 3}, {UINT64_MAX, 256, 1024, 0, 3},
                                   {UINT64_MAX, 256, 1024, 0, 4}};
    ResShape r{};
    for (const Shape &s : shapes) {
        if (g->m >= s.max_m) continue;
        const uint32_t groups = ((g->n - 1) >> s.lgK) + 1;
        r.W = s.W;
        while (r.W > 1 && r.W / 2 >= groups) r.W /= 2;
        r.bs = s.bs;
        r.lgK = s.lgK;
        r.one_xcd = r.W > 1 ? s.one_xcd : 0;
        const uint32_t per = r.W * r.bs, nj = (groups - 1) / per + 1;  // slots of every thread
        r.slots = nj * r.bs;
        r.fits = nj <= kMaxJ;
        if (r.fits) break;
    }
    r.bytes = ((sizeof(ResCtl) + 255) & ~255ull) + (uint64_t)r.W * (kShareCap * 16 + 2ull * r.slots) + 16ull * g->n;
    return r;
}

static ResArgs resident_args(const sssp_graph *g, const ResShape &r, uint32_t source, uint64_t *dist_out, void *scratch,
                             ResCtl **ctl) {
    ResArgs a;
    memset(&a, 0, sizeof a);
    a.rp = g->rp;
    a.edges = g->edges;
    a.vmin = g->vmin;
    a.emin = g->emin;
    a.dist = (unsigned long long *)dist_out;
    *ctl = (ResCtl *)scratch;
    a.bar = (*ctl)->bar;
    a.error = &(*ctl)->error;
    a.learn = &(*ctl)->learn;
    a.rec = (unsigned long long *)((uint8_t *)scratch + ((sizeof(ResCtl) + 255) & ~255ull));
    a.box = a.rec + 2ull * kShareCap * r.W;
    a.mark = (uint8_t *)(a.box + 2ull * g->n);
    a.share = g->max_deg > kShareDeg;
    a.quota = kQuota;
    a.n = g->n;
    a.max_phases = g->n;  // a phase settles at least the queue minimum
    a.polls = g->wait_polls ? g->wait_polls : kResSpin;
    a.m = g->m;
    a.src = source;
    a.wmax = g->wmax;
    a.W = r.W;
    a.lgW = (uint32_t)__builtin_ctz(r.W);
    a.lgK = r.lgK;
    a.lgWv = (uint32_t)__builtin_ctz((uint32_t)r.bs / 64);
    a.wslots = r.slots >> a.lgWv;
    a.mstride = r.slots;
    a.ip = g->ip;
    a.in_edges = g->in_edges;
    a.in_head = g->b.in_head;
    a.out_head = g->b.out_head;
    a.in_cur = g->b.in_cur;
    a.out_cur = g->b.out_cur;
    return a;
}

// Whether the resident form is the faster one. It saves about 10 us a phase or round, but relaxes a
// large set of edges more slowly than the phase kernels do, whose blocks take equal shares of it: where
// a solve has few and large phases they win. What tells is the mean weight (the smaller the weights,
// the fewer distances there are and the fewer phases) against the size m + 4 n, and whether a few
// rows hold many of the edges (`skewed`), which resident workgroups share only by records. Times of
// the resident form over the phase kernels', weights uniform in [1, w]:
//   static        R-MAT 22 (65 M edges)  w = 4  1.30, 64  1.07, 256  0.89;   R-MAT 21  w = 4  1.19, 16  0.93
//                 random, 67 M edges     w = 4  1.03 - 1.06, 16  0.94 - 0.97;   smaller graphs below 1 at any w
//   SIMPLE        R-MAT 22               w = 64  1.12, 256  0.97;   R-MAT 21  w = 4  1.24, 16  0.98
//                 random, 67 M edges     w = 16  0.96 - 1.08, 64  0.72 - 1.00;   34 M  w = 1  1.05, 4  0.95
//   checkpoint    (a pass counts the relaxations, a random load per edge)
//                 R-MAT 22               w = 2^14  1.06, 2^20  0.91;   R-MAT 20 and 21  w = 2^10  1.05 - 1.17, 2^14  0.96
//                 R-MAT 18, 8 M edges    w = 256  1.05, 1024  0.94
//                 random, 67 M edges     w = 64  1.15 - 1.23, 256  0.90 - 1.11;   34 M  w = 16  1.03, 64  0.93
//                 random of degree 64 and 200, 17 to 20 M edges  w = 16  1.17 - 1.23, 1024  0.73 - 0.87
//   Delta-stepping, by the width over the largest weight (a wide bucket is one large set)
//                 R-MAT 22               1/16  1.10, 1/32  0.76;   R-MAT 18 to 21, 4 to 32 M edges  1/4  1.02 - 1.11, 1/8  0.73 - 0.89
//                 R-MAT 14 and 16, 0.2 to 1 M edges  1/2  1.25, 1/4  0.84 - 0.95;   1  1.03 - 1.9, 1/2  0.84 - 1.25
//                 random of degree 64 and more, over 4 M edges  1  1.03 - 1.08, 1/2  0.81 - 0.88;   0.6 M edges  1/2  1.09, 1/4  0.85
bool resident_pays(const sssp_graph *g, int in, int out, uint64_t delta, bool learn) {
    if (g->m == 0) return true;
    // uniform weights lie in [1, w - 1]; all zero count as ones
    const double m = (double)g->m, n = g->n, w = std::max(2.0 * (double)g->sum_w / m, 1.0);
    const double size = m + 4 * n, million = 1e6;
    const bool skewed = g->max_deg > kShareDeg && g->max_deg > 8 * m / n, dense = m >= 48 * n;
    if (delta) {
        double wide = INFINITY;  // widths from here on, in parts of the largest weight
        if (skewed) wide = m >= 40 * million ? 0.05 : m >= 1 * million ? 0.2 : m >= 0.25 * million ? 0.4 : m >= 0.12 * million ? 0.75 : INFINITY;
        else if (dense && w > 16) wide = m >= 4 * million ? 0.75 : m >= 0.5 * million && m < 1 * million ? 0.4 : INFINITY;
        return (double)delta < wide * w;
    }
    double low = 0;  // weights up to here
    if (learn) {
        if (skewed) low = size >= 67 * million ? 20000 : size >= 15 * million ? 1500 : m >= 4 * million ? 400 : 0;
        else if (dense) low = m >= 4 * million ? 300 : 0;
        else low = size >= 67 * million ? 100 : size >= 25 * million ? 20 : m >= 16 * million ? 4 : 0;
    } else {
        const bool simple = in == IN_SIMPLE_M || out == OUT_SIMPLE_M;
        if (skewed) low = size >= 67 * million ? 100 : size >= 25 * million ? 6 : 0;
        else low = size >= 67 * million ? (simple ? 20 : 6) : size >= 25 * million && simple ? 2 : 0;
    }
    return w > low;
}

static dim3 vertex_grid(uint32_t n) {
    const uint64_t b = ((uint64_t)n + 255) / 256;
    return dim3((uint32_t)(b > 2048 ? 2048 : b < 64 ? 64 : b));
}

// *ran = false: the device cannot hold the workgroups at once.
static int resident_launch(rfn k, const ResShape &r, hipStream_t s, ResArgs a, ResCtl *ctl, size_t lds, bool *ran) {
    if (lds > 65536) HIP_OK(hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    uint32_t one_xcd = r.one_xcd;
    void *args[] = {&a, &ctl, &one_xcd};
    const hipError_t e = hipLaunchCooperativeKernel((const void *)k, dim3(r.one_xcd ? 8 * r.W : r.W), dim3(r.bs), args,
                                                    (uint32_t)lds, s);
    *ran = e != hipErrorCooperativeLaunchTooLarge;
    if (*ran) HIP_OK(e);
    else (void)hipGetLastError();
    return SSSP_OK;
}

// What a launch's error word says. 1: a workgroup waited too long for another, the solve is not
// finished (*ran = false). 2: more phases than there can be, unless the caller set the bound.
static int resident_verdict(unsigned int error, bool capped, bool *ran) {
    *ran = error == 0;
    if ((error & 2u) && !capped) return sssp_set_error(SSSP_ERR_INTERNAL, "a resident solve exceeded its phase bound");
    return SSSP_OK;
}

// Runs a resident solve (delta > 0: Delta-stepping) with `scratch` (r.bytes, 256-byte aligned).
// *ran = false: the device cannot hold the workgroups at once, one waited too long for another (the
// device is shared with other work), or it took more than `cap` phases (0: no cap); the distances are
// unfinished.
int resident_solve(const sssp_graph *g, const ResShape &r, hipStream_t s, uint32_t source, int in, int out, uint64_t delta,
                   uint64_t *dist_out, void *scratch, uint32_t *phases, bool *ran, uint32_t cap) {
    ResCtl *ctl;
    ResArgs a = resident_args(g, r, source, dist_out, scratch, &ctl);
    a.delta = delta;
    if (delta) a.max_phases = 4 * (g->n + 17);  // a bucket's light rounds each remove or lower
    if (cap) a.max_phases = cap;
    if (in == IN_SIMPLE_M || out == OUT_SIMPLE_M)
        hipLaunchKernelGGL(k_res_init_simple, vertex_grid(g->n), dim3(256), 0, s, a, ctl, (int)(in == IN_SIMPLE_M));
    else hipLaunchKernelGGL(k_res_init, vertex_grid(g->n), dim3(256), 0, s, a, ctl);
    const int rc = resident_launch(pick_res(r.bs, r.lgK, in, out, delta != 0), r, s, a, ctl, res_lds(r.slots, r.bs), ran);
    if (rc || !*ran) return rc;
    unsigned int h[2];
    static_assert(offsetof(ResCtl, phases) == offsetof(ResCtl, error) + 4, "one copy");
    HIP_OK(hipMemcpyAsync(h, &ctl->error, sizeof h, hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    *phases = h[1];
    return resident_verdict(h[0], cap != 0, ran);
}

// The static stage of a learned checkpoint solve, with scratch of resident_learn_bytes. Where the
// selector ends it, out->min_d is below INF64 and resident_learn_state has to follow. The phases take
// 8.9 us on a random graph of 1 M vertices and degree 16 (7.5 without the counts, whose atomics
// return a value; 17.8 with the phase kernels), so that a solve of 272 static phases and 22 others
// takes 4.1 ms, 6.2 before; one of 192 static phases on 100 k vertices 1.4 and 3.4.
uint64_t resident_learn_bytes(const sssp_graph *g, const ResShape &r) { return ((r.bytes + 255) & ~255ull) + 4ull * g->n; }

int resident_learn(const sssp_graph *g, const ResShape &r, hipStream_t s, uint32_t source, const float *mlp_w, double wm,
                   uint64_t *dist_out, void *scratch, ResLearned *out, bool *ran) {
    ResCtl *ctl;
    ResArgs a = resident_args(g, r, source, dist_out, scratch, &ctl);
    a.mlp_w = mlp_w;
    a.wm = wm;
    a.sp = (uint32_t *)((uint8_t *)scratch + ((r.bytes + 255) & ~255ull));
    a.mlp_lds = (uint32_t)((res_lds(r.slots, r.bs) + 15) & ~15ull);
    const rfn k = r.bs == 512 ? (r.lgK == 3 ? k_resident<512, 8, IN_STATIC_M, OUT_STATIC_M, false, true>
                                            : k_resident<512, 16, IN_STATIC_M, OUT_STATIC_M, false, true>)
                              : (r.lgK == 3 ? k_resident<1024, 8, IN_STATIC_M, OUT_STATIC_M, false, true>
                                            : k_resident<1024, 16, IN_STATIC_M, OUT_STATIC_M, false, true>);
    hipLaunchKernelGGL(k_res_init, vertex_grid(g->n), dim3(256), 0, s, a, ctl);
    const int rc = resident_launch(k, r, s, a, ctl, a.mlp_lds + kMlpParams * sizeof(float), ran);
    if (rc || !*ran) return rc;
    const uint64_t cb = (g->m / kCountEdges + 256) / 256;
    hipLaunchKernelGGL(k_learn_counts, dim3((uint32_t)(cb > 4096 ? 4096 : cb)), dim3(256), 0, s, a);
    static_assert(offsetof(ResCtl, phases) == offsetof(ResCtl, error) + 4 &&
                  offsetof(ResCtl, learn) == offsetof(ResCtl, error) + 8, "one copy");
    struct {
        unsigned int error, phases;
        ResLearn learn;
    } h;
    HIP_OK(hipMemcpyAsync(&h, &ctl->error, sizeof h, hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    const int rv = resident_verdict(h.error, false, ran);
    if (rv || !*ran) return rv;
    *out = h.learn.out;
    out->reached += 1;  // the source
    out->phases = h.phases;
    out->choice = (uint32_t)h.learn.choice[h.phases / 16 & 1];
    // those still queued have been so up to the last phase
    if (out->min_d != INF64) out->sum_f += (unsigned long long)out->phases * (out->reached - out->settled);
    return SSSP_OK;
}

// Where the selector ended the stage: state bytes, distances, heads and cursors as the phase kernels
// keep them, after the control block has been set.
int resident_learn_state(const sssp_graph *g, const ResShape &r, hipStream_t s, uint64_t *dist_out, void *scratch) {
    ResCtl *ctl;
    ResArgs a = resident_args(g, r, 0, dist_out, scratch, &ctl);
    a.sp = (uint32_t *)((uint8_t *)scratch + ((r.bytes + 255) & ~255ull));
    hipLaunchKernelGGL(k_learn_state, vertex_grid(g->n), dim3(256), 0, s, a, g->b.st, g->b.in_head, g->b.out_head, g->b.ctl);
    HIP_OK(hipGetLastError());
    return SSSP_OK;
}

// ---------------------------------------------------------------------------
// Batches: gangs of kGang workgroups of one XCD, each first one team of kGang for the largest
// queries; when those are taken it splits into teams of half the size for the next class, down to
// single workgroups. The smallest class whose lists fit LDS is the cheapest per query (a random
// graph of 16384 vertices, degree 16: 1.9 ms on one workgroup, 1.2 on two, 0.8 on four), so queries
// take it while there are more of them than workgroups, and larger teams when there is room. The
// longest query bounds a batch (a grid of 2^17 vertices takes 13.8 ms on eight workgroups, 12.5 on
// sixteen; giving such grids sixteen makes a batch of 192 queries 7 % faster and one of 512 14 %
// slower). 192 queries over 24 graphs up to 2^17 vertices: 18.2 ms, against 45.1 with one workgroup
// of 512 threads per query (batch.hip), 344 random and R-MAT queries up to 2^18 25 against 126. Grids
// in numbers that do not fit at once are for batch.hip (batch_split).
constexpr uint32_t kGangLog = 5, kGang = 1u << kGangLog;
constexpr int kBatchBs = 512;                    // threads: two workgroups per CU
constexpr uint32_t kBatchNj = 4;                 // slots per thread of a batch workgroup at most
constexpr uint32_t kWgVertices = 8u * kBatchBs * kBatchNj;  // vertices per workgroup at most
constexpr uint32_t kTeamBar = team_words(kGang) + kSlotStride;  // u64 of a team: its words, query word

struct ResQuery {
    const uint32_t *rp;
    const uint2 *edges;
    const uint2 *vmin;
    const uint32_t *emin;
    unsigned long long *dist;
    uint32_t n, src, wmax, share;
};

struct ResBatch {
    const ResQuery *q;
    const uint32_t *order;            // queries by class, the costliest first
    uint32_t first[kGangLog + 1], count[kGangLog + 1];
    uint32_t *heads;                  // queries taken, by class
    uint32_t *phases;
    unsigned int *error;
    unsigned long long *bar;          // 2 * kGang teams per gang
    unsigned long long *rec, *box;    // per workgroup: kShareCap records, 2 * wgv boxes
    uint8_t *mark;                    // per workgroup: 2 * slots
    uint32_t wgv, slots;
    uint32_t polls;                   // as in ResArgs
};

__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
template <typename T>
__device__ __forceinline__ T *uniform(T *p) {
    const unsigned long long x = (unsigned long long)p;
    return (T *)(((unsigned long long)uniform((uint32_t)(x >> 32)) << 32) | uniform((uint32_t)x));
}

template <int IN, bool OUT>
__global__ __launch_bounds__(kBatchBs, 4) void k_resident_batch(ResBatch b) {
    constexpr uint32_t BS = kBatchBs, K = 8, lgWv = 3;
    static_assert(BS / 64 == 1u << lgWv, "wavefronts");
    __shared__ uint32_t s_q, s_bad;
    const uint32_t tid = threadIdx.x;
    // workgroups are dealt out to the XCDs in turn: a gang's lie 8 apart, on one XCD
    const uint32_t gang = blockIdx.x / (8 * kGang) * 8 + blockIdx.x % 8, member = blockIdx.x / 8 % kGang;
    for (int cls = kGangLog; cls >= 0; --cls) {
        const uint32_t count = b.count[cls];
        if (count == 0) continue;  // grid-uniform
        const uint32_t W = 1u << cls, wg = member & (W - 1), m0 = member - wg;
        const uint64_t g0 = (uint64_t)gang * kGang + m0;  // the team's first workgroup
        unsigned long long *bar = b.bar + ((uint64_t)gang * 2 * kGang + (kGang >> cls) + (member >> cls)) * kTeamBar;
        unsigned long long *qword = bar + team_words(kGang);
        uint32_t nb = 0;
        for (uint32_t turn = 1;; ++turn) {
            // the team's first workgroup takes the next query and tells the others
            if (tid == 0) {
                uint32_t q = INF32;
                if (wg == 0) {
                    q = umin32(atomicAdd(&b.heads[cls], 1u), count);
                    if (W > 1) st_agent(qword, ((unsigned long long)turn << 32) | q);
                } else {
                    unsigned long long x = 0;
                    for (uint32_t spins = 0; spins < b.polls; ++spins) {
                        x = ld64(qword);
                        if ((uint32_t)(x >> 32) == turn) { q = (uint32_t)x; break; }
                        __builtin_amdgcn_s_sleep(1);
                    }
                }
                s_q = q;
                s_bad = 0;
            }
            __syncthreads();
            const uint32_t qi = uniform(s_q);
            if (qi == INF32) {
                if (tid == 0) atomicOr(b.error, 1u);
                return;
            }
            if (qi >= count) break;
            const uint32_t id = uniform(b.order[b.first[cls] + qi]);
            const ResQuery &rq = b.q[id];
            ResArgs a;
            a.rp = uniform(rq.rp);
            a.edges = uniform(rq.edges);
            a.vmin = uniform(rq.vmin);
            a.emin = uniform(rq.emin);
            a.dist = uniform(rq.dist);
            a.n = uniform(rq.n);
            a.src = uniform(rq.src);
            a.wmax = uniform(rq.wmax);
            a.share = uniform(rq.share);
            a.box = b.box + g0 * 2 * b.wgv;
            a.rec = b.rec + g0 * 2 * kShareCap;
            a.mark = b.mark + g0 * 2 * b.slots;
            a.bar = bar;
            a.error = b.error;
            a.W = W;
            a.lgW = (uint32_t)cls;
            a.lgWv = lgWv;
            a.lgK = 3;
            a.quota = kQuota;
            a.max_phases = a.n;
            a.polls = b.polls;
            a.delta = 0;
            const uint32_t groups = (a.n - 1) / K + 1;
            a.wslots = 64 * ((groups - 1) / (W * BS) + 1);
            a.mstride = a.wslots << lgWv;
            // this workgroup's groups: distances, boxes and marks
            for (uint32_t i = tid; i < a.mstride * K; i += BS) {
                const uint32_t v = (((i / K) << a.lgW) | wg) * K + i % K;
                if (v >= a.n) continue;
                const unsigned long long x = v == a.src ? 0ull : INF64;
                a.dist[v] = x;
                st_agent(&a.box[2ull * v], x);
                st_agent(&a.box[2ull * v + 1], x);
            }
            const uint64_t ms = mark_of(a, a.src / K);
            uint32_t *mw = reinterpret_cast<uint32_t *>(a.mark);
            for (uint32_t p = 0; p < 2; ++p)
                for (uint32_t i = tid; i < a.mstride / 4; i += BS) {
                    const uint64_t w = ((uint64_t)p * W + wg) * a.mstride / 4 + i;
                    st_agent(&mw[w], w == ms / 4 ? phase_tag(0) << (8 * (ms & 3)) : 0u);
                }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (W > 1) {  // the team's set-up is done
                unsigned long long *words = bar + bar_words(nb, W);
                const unsigned long long tag = bar_tag(nb);
                if (tid == 0) bar_put_empty(nb, W, wg, [&](uint32_t i, unsigned long long x) { st_agent(&bar[i], x); });
                ++nb;
                if (tid < W) {
                    uint32_t spins = 0;
                    while ((ld64(&words[tid * kSlotStride]) & kTag) != tag && ++spins < b.polls) {}
                    if (spins >= b.polls) s_bad = 1;
                }
                __syncthreads();
                if (s_bad) {  // block-uniform
                    if (tid == 0) atomicOr(b.error, 1u);
                    return;
                }
            }
            const uint32_t phases = resident_run<BS, K, IN, OUT, false>(a, wg, nb);
            if (phases == INF32) return;
            if (wg == 0 && tid == 0) b.phases[id] = phases;
            __syncthreads();  // LDS is set up anew for the next query
        }
        __syncthreads();
    }
}

typedef void (*bafn)(ResBatch);

static bafn pick_res_batch(int in, bool out) {
    if (in == IN_DIJK) return out ? k_resident_batch<IN_DIJK, true> : k_resident_batch<IN_DIJK, false>;
    if (in == IN_STATIC_M) return out ? k_resident_batch<IN_STATIC_M, true> : k_resident_batch<IN_STATIC_M, false>;
    return k_resident_batch<IN_NONE, true>;
}

static uint64_t up256(uint64_t x) { return (x + 255) & ~255ull; }

bool resident_batch_takes(const sssp_graph *g) { return g->n <= (uint64_t)kGang * kWgVertices; }
// The class of the least team whose lists hold the graph: it has 1 << class workgroups.
uint32_t resident_batch_class(const sssp_graph *g) {
    uint32_t c = 0;
    while (((uint64_t)kWgVertices << c) < g->n) ++c;
    return c;
}

// Whether a query's solve will take many phases, from what its source reaches in few hops: one
// workgroup per query walks up to kProbeHops hops and says so when they reached at most kProbeSeen
// vertices and did not run out. Grids and meshes of up to eight neighbours reach at most 1089 and take 5 to
// 21 sqrt(n) phases; random and R-MAT graphs, or grids in three dimensions, reach more and take at
// most 2.6 sqrt(n). A row of more than kProbeRow edges also means few phases. About 60 us for 512
// queries, with loads that wait for one another.
constexpr uint32_t kProbeHops = 16, kProbeSeen = 2048, kProbeRow = 256, kProbeSlots = 4 * kProbeSeen;
__global__ __launch_bounds__(256) void k_batch_probe(const ResQuery *q, uint32_t *many) {
    __shared__ uint32_t table[kProbeSlots], front[2][kProbeSeen];  // vertices seen (INF32: none), by hash; a hop's
    __shared__ uint32_t s_seen, s_next, s_few;
    const uint32_t tid = threadIdx.x;
    const ResQuery rq = q[blockIdx.x];
    for (uint32_t i = tid; i < kProbeSlots; i += 256) table[i] = INF32;
    if (tid == 0) {
        front[0][0] = rq.src;
        s_seen = 1;
        s_few = 0;
    }
    __syncthreads();
    // true if v was not there; at most kProbeSeen + 256 get in, so that there are free slots
    auto insert = [&](uint32_t v) {
        uint32_t i = v * 2654435769u >> 19;
        for (;;) {
            const uint32_t old = atomicCAS(&table[i], INF32, v);
            if (old == INF32 || old == v) return old == INF32;
            i = (i + 1) % kProbeSlots;
        }
    };
    static_assert(kProbeSlots == 1u << (32 - 19), "hash");
    if (tid == 0) insert(rq.src);
    uint32_t nf = 1;
    for (uint32_t hop = 0; hop < kProbeHops && nf; ++hop) {  // block-uniform
        __syncthreads();
        if (tid == 0) s_next = 0;
        __syncthreads();
        bool few = false;
        for (uint32_t j = tid; j < nf && !few; j += 256) {
            const uint32_t u = front[hop & 1][j], r0 = rq.rp[u], r1 = rq.rp[u + 1];
            few = r1 - r0 > kProbeRow;
            for (uint32_t e = r0; e < r1 && !few; ++e) {
                const uint32_t v = rq.edges[e].x;
                if (!insert(v)) continue;
                few = atomicAdd(&s_seen, 1u) >= kProbeSeen;  // each thread's last insertion then
                if (!few) front[(hop & 1) ^ 1][atomicAdd(&s_next, 1u)] = v;
            }
        }
        if (few) s_few = 1;
        __syncthreads();
        nf = s_few ? 0 : s_next;
    }
    if (tid == 0) many[blockIdx.x] = nf != 0;
}

// many[j] = the probe of query ids[j], with graphs[0]'s scratch on its stream.
int resident_probe(sssp_graph *const *graphs, const uint32_t *sources, const std::vector<uint32_t> &ids,
                   std::vector<uint32_t> *many) {
    const uint32_t nq = (uint32_t)ids.size();
    const uint64_t o_many = up256(nq * sizeof(ResQuery));
    const int rc = resident_scratch(graphs[0], o_many + 4ull * nq);
    if (rc) return rc;
    hipStream_t s = graphs[0]->stream;
    uint8_t *base = (uint8_t *)graphs[0]->res;
    std::vector<ResQuery> hq(nq);
    for (uint32_t j = 0; j < nq; ++j) {
        const sssp_graph *g = graphs[ids[j]];
        hq[j] = ResQuery{g->rp, g->edges, g->vmin, g->emin, nullptr, g->n, sources[ids[j]], g->wmax, 0u};
    }
    many->resize(nq);
    HIP_OK(hipMemcpyAsync(base, hq.data(), nq * sizeof(ResQuery), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_batch_probe, dim3(nq), dim3(256), 0, s, (const ResQuery *)base, (uint32_t *)(base + o_many));
    HIP_OK(hipGetLastError());
    HIP_OK(hipMemcpyAsync(many->data(), base + o_many, 4ull * nq, hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    return SSSP_OK;
}

// Solves the queries ids[0 .. nq) (each of a graph that resident_batch_takes) in one cooperative
// launch on graphs[0]'s stream and scratch. *ran = false: as in resident_solve, or no memory for it.
int resident_batch(sssp_graph *const *graphs, const uint32_t *sources, const uint32_t *ids, uint32_t nq, int in,
                   bool out_static, uint64_t *const *dist_outs, uint32_t *phases_out, bool *ran) {
    *ran = false;
    hipStream_t s = graphs[0]->stream;
    const bafn k = pick_res_batch(in, out_static);
    int dev = 0, cus = 0, per_cu = 0;
    HIP_OK(hipGetDevice(&dev));
    HIP_OK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // classes: the least team whose lists hold the graph, doubled while all queries fit at once
    std::vector<uint32_t> cls(nq);
    uint64_t wgs = 0;
    uint32_t slots = 0, wgv = 0;
    for (uint32_t i = 0; i < nq; ++i) {
        cls[i] = resident_batch_class(graphs[ids[i]]);
        wgs += 1u << cls[i];
    }
    auto lds_slots = [&](uint32_t n, uint32_t c) { return kBatchBs * ((((n - 1) / 8 + 1) - 1) / (kBatchBs << c) + 1); };
    for (uint32_t i = 0; i < nq; ++i) slots = std::max(slots, lds_slots(graphs[ids[i]]->n, cls[i]));
    HIP_OK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k, kBatchBs, res_lds(slots, kBatchBs)));
    const uint64_t resident = (uint64_t)per_cu * cus / (8 * kGang) * (8 * kGang);
    if (resident == 0) return SSSP_OK;
    for (bool grown = true; grown && 2 * wgs <= resident;) {
        grown = false;
        for (uint32_t i = 0; i < nq; ++i)
            // at least a slot per thread of work
            if (cls[i] < kGangLog && (4096u << cls[i]) <= graphs[ids[i]]->n) {
                wgs += 1u << cls[i]++;
                grown = true;
            }
    }
    slots = 0;
    for (uint32_t i = 0; i < nq; ++i) {
        slots = std::max(slots, lds_slots(graphs[ids[i]]->n, cls[i]));
        wgv = std::max(wgv, 8 * ((((graphs[ids[i]]->n - 1) / 8 + 1) - 1) / (1u << cls[i]) + 1));
    }
    const uint64_t blocks = std::min(resident, (wgs + 8 * kGang - 1) / (8 * kGang) * (8 * kGang));
    const uint64_t gangs = blocks / kGang;
    // costliest first: a graph of low degree takes the most phases for its size (a grid of 2^17
    // vertices 2946, a random graph of degree 16 207)
    auto cost = [&](uint32_t i) {
        const sssp_graph *g = graphs[ids[i]];
        return g->m < 6ull * g->n ? 16ull * g->n : (uint64_t)g->n + g->m / 8;
    };
    std::vector<uint32_t> order(nq);
    for (uint32_t i = 0; i < nq; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
        return cls[x] != cls[y] ? cls[x] > cls[y] : cost(x) > cost(y);
    });
    ResBatch b;
    memset(&b, 0, sizeof b);
    for (uint32_t i = 0; i < nq; ++i) ++b.count[cls[i]];
    for (int c = kGangLog - 1; c >= 0; --c) b.first[c] = b.first[c + 1] + b.count[c + 1];
    // one buffer: [queries, order | heads, error | phases | barrier words | records | boxes | marks]
    const uint64_t o_order = up256(nq * sizeof(ResQuery)), o_heads = up256(o_order + 4ull * nq),
                   o_phases = up256(o_heads + 4 * (kGangLog + 2)), o_bar = up256(o_phases + 4ull * nq),
                   o_rec = up256(o_bar + gangs * 2 * kGang * kTeamBar * 8), o_box = up256(o_rec + blocks * kShareCap * 16),
                   o_mark = up256(o_box + blocks * wgv * 16), total = o_mark + blocks * 2 * slots;
    // kept on graphs[0]: allocating and freeing it took 0.4 to 8 ms a call
    const int rc = resident_scratch(graphs[0], total);
    if (rc) return rc == SSSP_ERR_OOM ? SSSP_OK : rc;
    uint8_t *base = (uint8_t *)graphs[0]->res;
    std::vector<uint8_t> up(o_heads);
    ResQuery *hq = (ResQuery *)up.data();
    for (uint32_t i = 0; i < nq; ++i) {
        const sssp_graph *g = graphs[ids[i]];
        hq[i] = ResQuery{g->rp, g->edges, g->vmin, g->emin, (unsigned long long *)dist_outs[ids[i]],
                         g->n, sources[ids[i]], g->wmax, g->max_deg > kShareDeg};
    }
    memcpy(up.data() + o_order, order.data(), 4ull * nq);
    HIP_OK(hipMemcpyAsync(base, up.data(), o_heads, hipMemcpyHostToDevice, s));
    HIP_OK(hipMemsetAsync(base + o_heads, 0, o_rec - o_heads, s));
    b.q = (const ResQuery *)base;
    b.order = (const uint32_t *)(base + o_order);
    b.heads = (uint32_t *)(base + o_heads);
    b.error = b.heads + kGangLog + 1;
    b.phases = (uint32_t *)(base + o_phases);
    b.bar = (unsigned long long *)(base + o_bar);
    b.rec = (unsigned long long *)(base + o_rec);
    b.box = (unsigned long long *)(base + o_box);
    b.mark = base + o_mark;
    b.wgv = wgv;
    b.slots = slots;
    b.polls = graphs[0]->wait_polls ? graphs[0]->wait_polls : kResSpin;
    const size_t lds = res_lds(slots, kBatchBs);
    if (lds > 65536) HIP_OK(hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    void *args[] = {&b};
    const hipError_t e = hipLaunchCooperativeKernel((const void *)k, dim3((uint32_t)blocks), dim3(kBatchBs), args,
                                                    (uint32_t)lds, s);
    if (e == hipErrorCooperativeLaunchTooLarge) {
        (void)hipGetLastError();
        return SSSP_OK;
    }
    HIP_OK(e);
    std::vector<uint32_t> down((o_bar - o_heads) / 4);
    HIP_OK(hipMemcpyAsync(down.data(), base + o_heads, o_bar - o_heads, hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    const int rv = resident_verdict(down[kGangLog + 1], false, ran);
    if (rv == SSSP_OK && *ran && phases_out)
        for (uint32_t i = 0; i < nq; ++i) phases_out[ids[i]] = down[(o_phases - o_heads) / 4 + i];
    return rv;
}
