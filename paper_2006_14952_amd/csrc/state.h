// The opaque tree handle: every device buffer of one box, grown on demand.
#pragma once
#include <vector>

#include "common.h"
#include "p2p_law.h"

namespace hfmm {
constexpr int kHostInts = 4096;
// Interaction list kinds: 0 M2L, 1 P2P, 2 handed to the children, 3 candidate pairs
// (training export), 4 M2L pairs of the learned selector (all orders; the order of each
// entry in a byte beside it).
constexpr int kKinds = 5;
constexpr int kKindCand = 3, kKindOrd = 4;
constexpr int kOrders = 7;  // learned selector: M2L orders 2 .. 8

// Device counters of one evaluation (fmm_tree::counters), in bytes from its start:
//   kErrByte    int: the traversal's overflow bits
//   kPoolByte   chunk counters of the list kinds, one 128-byte line each
//   kTravByte   kTravSlots lines of 64-bit sums of the traversal: visits, M2L pairs, P2P
//               pairs, M2L pairs of each learned order, largest P2P leaf; the readback ends
//               after them
//   kP2PByte    kP2PSlots lines of 64-bit sums of P2P: listed pairs, evaluated pairs
// Atomics on one address end one after the other, about 13 ns apart on this GPU: with one
// address per sum, a 4096-wave traversal launch took 160 us whatever its work (three sums a
// wave) and P2P of 4096 leaves 106 us of its 160.  A wave adds to the line of its
// workgroup's number, and the host sums the lines.  Traversal of the 2M box 1.84 -> 1.04 ms, with the
// learned selector (ten sums a wave) 2.90 -> 1.16, of 262,144 particles 1.15 -> 0.52.
constexpr int kErrByte = 96;
constexpr int kPoolByte = 256;
constexpr int kPoolStride = 32;  // ints between the pool counters
constexpr int kSlotWords = 16;   // 64-bit words per line
constexpr int kTravSlots = 64, kP2PSlots = 256;
constexpr int kTravByte = kPoolByte + kKinds * kPoolStride * 4;
constexpr int kP2PByte = kTravByte + kTravSlots * kSlotWords * 8;
constexpr int kCounterBytes = kP2PByte + kP2PSlots * kSlotWords * 8;
static_assert(kP2PByte <= kHostInts * 4, "counter readback exceeds the pinned area");
}

struct fmm_tree {
    // shape
    int64_t n = 0;
    double box = 1.0;
    int ncrit = 32;
    int ncell = 0, nleaf = 0, nlevel = 0;  // levels 0 .. nlevel-1 are non-empty
    int nbox = 1;                          // roots: one per box of a batch
    std::vector<int> hboxoff;              // particle offsets of the boxes (host copy)
    std::vector<int> lvl_beg;              // cells of level l: lvl_beg[l] .. lvl_beg[l+1]-1
    std::vector<int> leaf_lvl;             // leaves of level l: leaves[leaf_lvl[l] .. leaf_lvl[l+1]-1]

    // particles, Morton order
    hfmm::DevBuf keys[2], idx[2];
    int sorted = 0;               // which of keys/idx holds the sorted order
    hfmm::DevBuf boxoff;          // int[nbox + 1] particle offsets of the boxes
    hfmm::DevBuf xs, ys, zs, ms;  // wrapped FP64 positions and masses
    hfmm::DevBuf perm;            // sorted index -> caller index
    hfmm::DevBuf leaf_of;         // sorted index -> leaf cell
    hfmm::DevBuf rel32;           // float4 (x - c_leaf, m) for the FP32 form
    hfmm::DevBuf nearf;           // near-field acceleration, 3 x n FP64 (SoA)

    // cells
    hfmm::DevBuf cells;           // Cell[ncell]
    hfmm::DevBuf leaves;          // int[nleaf]
    hfmm::DevBuf inner;           // int[ncell - nleaf]: the cells with children, level by level
    hfmm::DevBuf Mc, Lc;          // expansion coefficients, ncell x ncoef(p) (float or double)

    // interaction lists: per cell and list kind (hfmm::kKinds), a chain of 64-entry chunks;
    // head[k * ncell + c], cnt[k * ncell + c].  lcnt continues with the learned selector's
    // per-order counts, cnt[(kKinds + o - 2) * ncell + c] for order o.
    hfmm::DevBuf lhead, lcnt;
    hfmm::DevBuf litems[hfmm::kKinds], lnext[hfmm::kKinds];
    hfmm::DevBuf lord;                               // kind kKindOrd: the M2L order of each entry (byte)
    int lcap[hfmm::kKinds] = {0};                    // chunks (one more is allocated as overflow bin)
    int64_t lseg[hfmm::kOrders] = {0};               // learned: start of each order's pairs in m2l_pairs
    int trav_mode = 0;                               // mode of the last traversal
    hfmm::DevBuf tstack;                             // per-wave traversal stacks
    hfmm::DevBuf cellc;                              // packed 16-byte cell view for the traversal
    int stk_cap = 4096;                              // entries per wave (grows on overflow)
    int64_t n_m2l = 0, n_p2p = 0, n_visit = 0, p2p_pairs = 0;
    int64_t p2p_max_cost = 0;                        // most list entries x passes of one sink leaf
    hfmm::P2PLaw64 law64;                            // FP64 P2P: the force law's constants
    hfmm::DevBuf p2p_wide;                           // sink leaves computed by workgroups of several waves
    hfmm::DevBuf counters;                           // device counters

    // scratch
    hfmm::DevBuf scan_tmp, nch, flag;
    hfmm::DevBuf m2l_ctr, m2l_pairs;  // flattened M2L pairs (sink, item) for the pair kernel; its fill counter
    hfmm::DevBuf wstate;              // per traversal wave: chunk block in use of each list kind
    hfmm::DevBuf bbox;                // per cell: float4 lo, hi of its particles relative to the centre (leaves)
    // matrix-core M2L: per cell the entries it takes (ne) and the others (no), their
    // offsets, the sinks with such entries (compacted), the entries by sink (CSR), totals
    hfmm::DevBuf mf_ne, mf_no, mf_offe, mf_offn, mf_spos, mf_sinks, mf_csr, mf_tot;
    int64_t mf_n_other = 0;           // sizes of the last split (a recorded replay reuses them)
    int mf_nsink = 0;
    hfmm::DevBuf cfeat;               // learned selector: per-cell part of the features (float4)
    int *host = nullptr;  // pinned readback area (kHostInts ints)
    int last_p = -1, last_prec = -1;

    // second stream (default priority) for stages independent of the caller's stream
    hipStream_t aux = nullptr;
    hipEvent_t dep[4]{};
    uint64_t pm_call = 0;                   // hybrid step: the long-range part's number
    hipEvent_t bev = nullptr;               // tree build: its sizes are in t->host
    // traversal: the lists of level l's sinks are complete (lev); P2P launch of level l (timing)
    hipEvent_t lev[hfmm::kMaxLevel + 1]{}, p2p_t0[hfmm::kMaxLevel + 1]{}, p2p_t1[hfmm::kMaxLevel + 1]{};
    bool lev_ready = false;

    // recorded evaluation (fmm_short_range_forces_graph): the executable graph, what it was
    // recorded with, and the build it belongs to
    hipGraphExec_t gexec = nullptr;
    fmm_params gparams{};
    double *gacc = nullptr;
    hipStream_t gstream = nullptr;
    uint64_t build_serial = 0, gserial = 0, gmoves = 0;
    int64_t g_n_m2l = 0, g_n_p2p = 0, g_n_visit = 0;  // the recorded evaluation's counts
    int64_t g_by_order[hfmm::kOrders] = {0};
    uint64_t gmodel = 0;                              // selector model the graph was recorded with
    bool capturing = false;  // run_forces is being recorded: no host reads, no timing

    // timing
    int timing = 0;
    fmm_stats stats{};
    hipEvent_t ev[16]{};
    bool events_ready = false;
};

namespace hfmm {
// Particles ordered by their Morton keys' leading bits (morton_order), with its buffers.
struct MortonSort {
    DevBuf keys[2], idx[2], xs, ys, zs, ms, tmp, scan_tmp;
    int sorted = 0;  // the pair of keys and idx (sorted -> caller index) in order
};
int morton_order(MortonSort &s, int n, double box, const double *pos, const double *mass, int levels, int *bad,
                 hipStream_t st);
int tree_build(fmm_tree *t, const fmm_params *P, int64_t n, const double *pos, const double *mass, int nbox,
               const int64_t *offsets, hipStream_t st);
// Called by the traversal after it has launched the kernel of sink level l on st: once that
// launch ends, the lists of the level's sinks are complete.  `side` is the stream the hook
// launches on; the traversal synchronises it before a rerun (whose lists replace these).
struct TravHook {
    int (*level)(void *ctx, int l, hipStream_t st);
    void *ctx;
    hipStream_t side;
};
int traverse(fmm_tree *t, const fmm_params *P, hipStream_t st, const TravHook *hook = nullptr);
struct MacModel;
int traverse_mode(fmm_tree *t, const fmm_params *P, int mode, double theta_max, const void *M, int mstride,
                  int mprec, const MacModel *model, hipStream_t st, const TravHook *hook = nullptr);
int upward(fmm_tree *t, const fmm_params *P, hipStream_t st);
int m2l(fmm_tree *t, const fmm_params *P, hipStream_t st);
int m2l_learned(fmm_tree *t, const fmm_params *P, hipStream_t st);
int downward_l2l(fmm_tree *t, const fmm_params *P, hipStream_t st);
// P2P of every sink leaf costing less than `line`; p2p_wide selects the others for workgroups
// of several waves (line: 2^62 if there are none) and p2p_wide_launch computes them
int p2p(fmm_tree *t, const fmm_params *P, long long line, hipStream_t st);
int p2p_wide(fmm_tree *t, const fmm_params *P, hipStream_t st, long long *line);
int p2p_wide_launch(fmm_tree *t, const fmm_params *P, long long line, hipStream_t st);
int p2p_tile(const fmm_params *P);  // sink particles per pass over a leaf's list
// P2P of the sink leaves leaves[first .. first+count-1]; with err non-NULL the launch does
// nothing while *err is non-zero (lists of a traversal that overflowed)
int p2p_range(fmm_tree *t, const fmm_params *P, int first, int count, const int *err, hipStream_t st);
int p2p_bbox(fmm_tree *t, const fmm_params *P, hipStream_t st);  // before p2p: leaf boxes
bool fused_applies(const fmm_params *P);                            // schedule 2 serves these parameters
int p2p_m2l_fused_prepare(fmm_tree *t, const fmm_params *P, hipStream_t st);  // schedule 2: L, pairs, queue
int p2p_m2l_fused_launch(fmm_tree *t, const fmm_params *P, hipStream_t st);   // P2P + M2L, one launch
int l2p_combine(fmm_tree *t, const fmm_params *P, double *acc, int accumulate, hipStream_t st);
// FP32 M2L of order p in 4..8 on the matrix cores for pairs on one level; the other
// pairs are left in t->m2l_pairs, their number in *n_other (L zeroed by the caller)
int m2l_mfma_split_and_run(fmm_tree *t, int p, Split sp, int64_t *n_other, hipStream_t st);
uint64_t cell_key_host(int level, int ix, int iy, int iz);
}  // namespace hfmm
