// The opaque sssp_graph handle and the helpers shared between translation units.
#pragma once

#include <vector>

#include "common.h"

struct sssp_graph {
    uint32_t n = 0;
    uint64_t m = 0;
    int device = 0;
    hipStream_t stream = nullptr;
    void *base = nullptr;          // the allocation that holds rp, edges, vmin and emin
    uint64_t base_bytes = 0;
    uint32_t *rp = nullptr;        // row_ptr as u32 (n+1)
    uint2 *edges = nullptr;        // (target, weight); rows sorted by weight once rows_sorted
    bool rows_sorted = false;      // set by graph_ensure_sorted (the dynamic criteria's cursors)
    uint2 *vmin = nullptr;         // (minIn, minOut)
    uint32_t *emin = nullptr;      // per edge: minOut of its target (relax folds the next OUT-STATIC threshold)
    uint32_t *ip = nullptr;        // CSC in_ptr (lazy)
    uint2 *in_edges = nullptr;     // CSC (source, weight), rows sorted by weight (lazy)
    uint64_t precompute_ns = 0;
    uint64_t sum_w = 0;            // exact sum of edge weights (selector feature scale)
    uint32_t max_deg = 0;          // longest row
    uint32_t wmax = 0;             // some edge weighs 2^32 - 1 (a stored minimum INF32 is then ambiguous)
    LaunchCfg cfg{};
    // per-solve scratch, allocated on first use and kept
    SolveBufs b{};
    bool bufs_ready = false;
    uint32_t bufs_scan_blocks = 0; // scan grid the S' shard capacity was sized for
    uint32_t delta_cap = 0;        // entries of b.deltas
    CtlHead *h_ctl = nullptr;      // pinned host mirror of the control-block header (2 slots)
    hipEvent_t ev[2] = {nullptr, nullptr};
    // per-kernel event timing
    bool prof = false;
    hipEvent_t *pev = nullptr;     // 4 events per phase of one batch
    uint32_t pev_cap = 0;
    sssp_kernel_profile last_prof{};
    std::vector<float> phase_ms;   // per-phase kernel time of the last timed solve
    // captured phase batch (6 phases) for graph replay
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    unsigned char graph_key[512] = {0};
    uint32_t graph_key_len = 0;
    // one-workgroup solves (launch option `single`): the batched kernel's per-query scratch
    uint8_t *one_st = nullptr;     // state bytes, n rounded up to 256
    uint32_t *one_fl = nullptr;    // two fringe lists and the settled list, 3 * n
    uint2 *one_fm = nullptr;       // (minIn, minOut) of the two fringe lists' entries, 2 * n
    void *one_aux = nullptr;       // query record, order, phase count, work-queue control
    uint32_t wait_polls = 0;       // longest wait of a resident workgroup (0: the default)
    uint32_t form = SSSP_FORM_NONE;  // what served the last solve
    // resident solves: barrier words and group marks
    void *res = nullptr;
    uint64_t res_bytes = 0;
};

DevGraph dev_view(const sssp_graph *g);
int graph_ensure_csc(sssp_graph *g);
int resident_scratch(sssp_graph *g, uint64_t bytes);
bool resident_release(sssp_graph *g);
int graph_ensure_sorted(sssp_graph *g);
void graph_default_cfg(sssp_graph *g);
int solve_bufs_ensure(sssp_graph *g, bool cursors, bool stamps, bool queue, bool approx = false, bool store = false);
void solve_bufs_free(sssp_graph *g);
int batch_solve_one(sssp_graph *g, uint32_t source, int in, bool out_static, uint64_t *dist_out,
                    uint32_t *phases_out);

// Shape of a resident solve (resident.hip).
struct ResShape {
    uint32_t W;           // workgroups (a power of two)
    uint32_t lgK;         // vertices per group: 8 or 16
    uint32_t slots;       // vertex groups a workgroup can hold
    uint32_t one_xcd;     // all workgroups on one XCD
    int bs;               // threads per workgroup
    bool fits;            // the graph can be solved resident
    uint64_t bytes;       // device scratch
};
ResShape resident_shape(const sssp_graph *g);
bool resident_pays(const sssp_graph *g, int in, int out, uint64_t delta, bool learn);
int resident_solve(const sssp_graph *g, const ResShape &r, hipStream_t s, uint32_t source, int in, int out, uint64_t delta,
                   uint64_t *dist_out, void *scratch, uint32_t *phases, bool *ran, uint32_t cap = 0);
// What the static stage of a learned checkpoint solve leaves: counts, and minD and the OUT-STATIC
// threshold of the phase after it (INF64: the solve is finished).
struct ResLearned {
    unsigned long long min_d, t, reached, settled, sum_f, m_reach, improving, relax_edges;
    uint32_t phases, choice;
};
uint64_t resident_learn_bytes(const sssp_graph *g, const ResShape &r);
int resident_learn(const sssp_graph *g, const ResShape &r, hipStream_t s, uint32_t source, const float *mlp_w, double wm,
                   uint64_t *dist_out, void *scratch, ResLearned *out, bool *ran);
int resident_learn_state(const sssp_graph *g, const ResShape &r, hipStream_t s, uint64_t *dist_out, void *scratch);
bool resident_batch_takes(const sssp_graph *g);
uint32_t resident_batch_class(const sssp_graph *g);
int resident_probe(sssp_graph *const *graphs, const uint32_t *sources, const std::vector<uint32_t> &ids,
                   std::vector<uint32_t> *many);
int resident_batch(sssp_graph *const *graphs, const uint32_t *sources, const uint32_t *ids, uint32_t nq, int in,
                   bool out_static, uint64_t *const *dist_outs, uint32_t *phases_out, bool *ran);
// A resident solve where the graph and its launch options allow one (phased.hip).
int resident_try(sssp_graph *g, uint32_t source, int in, int out, uint64_t delta, uint64_t *dist_out,
                 uint32_t *phases_out, bool *ran);
