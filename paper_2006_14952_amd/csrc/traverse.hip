// Dual tree traversal with the modified multipole acceptance criterion (Sec. 2.3).
//
// The dual traversal from the root pairs visits a cell pair (A, B) iff its parent pair
// was opened, and every decision depends on (A, B, image) alone.  It can therefore be
// run sink level by sink level: the pairs that a sink A meets are those its parent
// handed down ("open the sink"), expanded on the source side ("open the source").
// Each sink emits its M2L sources, its P2P sources (both leaves) and the pairs it hands
// to its children.  The set of pairs is exactly that of the recursive traversal.
//
// GPU form: one 64-lane wave per sink; a level's sinks are dealt round robin to a grid of
// as many waves as fit on the device at once.
// The wave takes up to 64 pending pairs at a time, decides them in parallel, appends
// the emitted pairs with ballots, and pushes opened sources' children on a per-wave
// stack (last in, first out).  Lists are chains of 64-entry chunks taken from pools
// with an atomic counter, so one pass and no host round trip per level is needed; a
// pool or stack that runs out is detected (the counter keeps the exact demand) and the
// traversal is rerun with enough room.  Per-sink list order is deterministic.
//
// Bound by the length of a step (64 pairs) in the waves with the heaviest sinks: a level ends
// with its longest wave, and more waves per SIMD do not shorten it (4, 6 and 8 measured
// alike).  So a step is kept short: the top of the stack and the open ends of the lists lie in
// LDS, whose accesses of one wave stay in order without waits, a list chunk leaves as one
// store when it is full, and the acceptance criterion runs on whole numbers in FP32.
// Traversal against pushes to device memory and FP64 decisions: 2M box 1.14 -> 0.78 ms, 64-box
// forest 1.55 -> 1.10, 16.7M 2.64 -> 1.96, 262,144 particles 0.61 -> 0.50, 2M learned 1.20 -> 1.03.
#include <math.h>
#include <string.h>

#include "mlp.h"
#include "state.h"

namespace hfmm {

// 0 = neglect (item 1), 1 = M2L (item 2), 2 = open (item 3 or item 2 failed).
// Distances are integers in units of u = box / 2^(l+1), l the finer level: every
// separation is below 2^23 and every squared distance below 2^50, so double precision
// holds them exactly and the comparisons are exact.
__device__ __forceinline__ int mac_decide(int4 a, int4 b, int s, const MacConst &mc)
{
    int la = xln_level(a.x), lb = xln_level(b.x);
    int l = la > lb ? la : lb;
    double wa = (double)(1 << (l - la)), wb = (double)(1 << (l - lb));
    double half = wa + wb, img = (double)(2 << l);
    double sh0 = (double)(s / 9 - 1), sh1 = (double)((s / 3) % 3 - 1), sh2 = (double)(s % 3 - 1);
    double R0 = (2.0 * xln_ix(a.x) + 1.0) * wa - (2.0 * xln_ix(b.x) + 1.0) * wb - sh0 * img;
    double R1 = (2.0 * a.y + 1.0) * wa - (2.0 * b.y + 1.0) * wb - sh1 * img;
    double R2 = (2.0 * a.z + 1.0) * wa - (2.0 * b.z + 1.0) * wb - sh2 * img;
    double A0 = fabs(R0), A1 = fabs(R1), A2 = fabs(R2);
    double g0 = fmax(A0 - half, 0.0), g1 = fmax(A1 - half, 0.0), g2 = fmax(A2 - half, 0.0);
    double sm2 = g0 * g0 + g1 * g1 + g2 * g2;
    double cut2 = ldexp(mc.cut2, 2 * l);  // equals (r_cut / u_l)^2 exactly
    double sc2 = R0 * R0 + R1 * R1 + R2 * R2;
    if (!(mc.mode & 4)) {  // truncated MAC; mode bit 2: conventional MAC, item 2 alone
        if (sm2 > cut2) return 0;
        double G0 = A0 + half, G1 = A1 + half, G2 = A2 + half;
        double sM2 = G0 * G0 + G1 * G1 + G2 * G2;
        bool straddle = (mc.mode & 1) ? (sc2 > cut2) : (sM2 > cut2);
        if (straddle) return 2;
    }
    double w = (mc.mode & 2) ? wb : fmax(wa, wb);
    if (4.0 * w * w <= mc.theta2 * sc2) return 1;
    return 2;
}

// Traversal modes: plain MAC; plain MAC plus export of candidate pairs; learned selector.
enum { kModePlain = 0, kModeExport = 1, kModeLearned = 2 };

struct TravArgs {
    const Cell *cells;
    int lbeg, ln, ncell;
    uint32_t *items[kKinds];
    int *next[kKinds];
    int cap[kKinds];
    int *pool;       // chunk counter of list kind k at pool[k * kPoolStride] (chunks handed out)
    int *wstate;     // per wave w: [kKinds] next chunk, [kKinds] end of its block, kept across levels
    int *head, *cnt; // [kKinds][ncell]
    unsigned char *ord;  // kind kKindOrd: the M2L order of each entry
    int *ocnt;           // learned: entries of order o of sink c at ocnt[(o - 2) * ncell + c]
    uint32_t *stack; // per-wave stacks when they do not fit in LDS
    int stk_cap;
    int *err;        // bit 0: stack overflow, bit 1: pool overflow
    // kTravSlots lines: [0] visits, [1] M2L, [2] P2P, [3 ..] M2L of each learned order, last the
    // most P2P entries times passes (of `tile` sink particles) of one leaf
    unsigned long long *slots;
    int tile;
    // candidate pairs / learned selector
    double theta_max2;             // candidates have (L/S_c)^2 <= theta_max2
    double box, rs, rcut;
    const float4 *cf;              // learned: per-cell part of the features (cell_features)
    const MacModel *model;
    const int4 *cellc;  // the first 16 bytes of every cell, packed (what the traversal reads)
};

constexpr int kChunkBlock = 32;   // chunks taken from a pool per atomic
constexpr int kCandQ = 128;       // learned: ring of candidate pairs (at most 63 wait between steps)

// A list being written: its first and latest chunk and its entries so far.  The entries past
// the last full chunk wait in an LDS ring of two chunks (slot = entry mod 128).
struct ListState {
    int head, cur, tot;
};
struct ListRing {
    uint32_t item[2 * kChunk];
};

// Orders the LDS accesses of one wave for the compiler; the hardware keeps them in order.
__device__ __forceinline__ void lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Next free chunk of list k.  Each wave takes kChunkBlock chunks per atomic and hands
// them out itself; the unused rest of its block passes to the wave with the same index
// in the next level's launch.  So the counters see one atomic per kChunkBlock chunks and
// no burst when a level starts (same-address atomics are serialised in the L2).  All
// list state is wave-uniform and kept in scalar registers.
__device__ __forceinline__ int new_chunk(const TravArgs &a, int k, int *bnext, int *bend, int lane)
{
    if (bnext[k] == bend[k]) {
        int c = 0;
        if (lane == 0) c = atomicAdd(&a.pool[k * kPoolStride], kChunkBlock);
        c = __builtin_amdgcn_readfirstlane(c);
        bnext[k] = c;
        bend[k] = c + kChunkBlock;
    }
    int c = bnext[k]++;
    if (c >= a.cap[k]) {  // out of room: write into the spare chunk, report, rerun later
        if (lane == 0) atomicOr(a.err, 2);
        c = a.cap[k];
    }
    return c;
}

// Write entries [first, first + n) of list k (a chunk's worth, n <= 64) from its ring.  ORD:
// with the byte beside each entry (list kind kKindOrd).
template <bool ORD>
__device__ __forceinline__ void flush(const TravArgs &a, int k, ListState &L, const ListRing &ring,
                                      const unsigned char *ordring, int *bnext, int *bend, int first, int n, int lane)
{
    const int c = new_chunk(a, k, bnext, bend, lane);
    if (L.cur < 0) L.head = c;
    else if (lane == 0) a.next[k][L.cur] = c;
    L.cur = c;
    if (lane < n) {
        const int at = (first + lane) & (2 * kChunk - 1);
        a.items[k][(size_t)c * kChunk + lane] = ring.item[at];
        if (ORD) a.ord[(size_t)c * kChunk + lane] = ordring[at];
    }
}

// Append `item` of every lane with `pred` to list k, in lane order.  A chunk is taken when
// 64 entries are there (or at the sink's end), so a chain never ends in an empty chunk.
template <bool ORD = false>
__device__ __forceinline__ void emit(const TravArgs &a, int k, ListState &L, ListRing &ring, unsigned char *ordring,
                                     int *bnext, int *bend, bool pred, uint32_t item, uint64_t lt, int lane,
                                     unsigned char ob = 0)
{
    const uint64_t mask = __ballot(pred);
    if (mask == 0) return;
    const int at = (L.tot + __popcll(mask & lt)) & (2 * kChunk - 1);
    if (pred) {
        ring.item[at] = item;
        if (ORD) ordring[at] = ob;
    }
    const int old = L.tot;
    L.tot += __popcll(mask);
    if ((L.tot ^ old) & ~(kChunk - 1)) {  // a chunk is full (64 entries at most were added)
        lds_order();
        flush<ORD>(a, k, L, ring, ordring, bnext, bend, old & ~(kChunk - 1), kChunk, lane);
        lds_order();
    }
}

// Full MAC evaluation for the candidate logic: code as mac_decide, plus whether the pair is a
// candidate of the selector (not neglected, not forced open by item 3, (L / S_c)^2 <= theta_max2).
struct MacEval {
    int code;
    bool cand;
};

__device__ __forceinline__ MacEval mac_eval(int4 a, int4 b, int s, const MacConst &mc, double theta_max2)
{
    MacEval r{0, false};
    PairGeo g = pair_geo(a, b, s);
    double cut2 = ldexp(mc.cut2, 2 * g.l);
    double w = (mc.mode & 2) ? g.wb : fmax(g.wa, g.wb);
    if (!(mc.mode & 4)) {  // truncated MAC; mode bit 2: conventional MAC, item 2 alone
        if (g.sm2 > cut2) return r;
        if ((mc.mode & 1) ? (g.sc2 > cut2) : (g.sM2 > cut2)) {
            r.code = 2;
            return r;
        }
    }
    r.code = (4.0 * w * w <= mc.theta2 * g.sc2) ? 1 : 2;
    r.cand = 4.0 * w * w / g.sc2 <= theta_max2;
    return r;
}

// The same decisions in FP32 on whole numbers (mc.whole): coordinates and distances are below
// 2^23, a squared distance that decides is below 2^24, and a larger one, though rounded, stays
// above every threshold.  tab: the three threshold tables.
__device__ __forceinline__ MacEval mac_whole(int4 a, int la, int4 b, int s, int mode, const float (*tab)[kMaxLevel + 1])
{
    const int lb = xln_level(b.x), l = max(la, lb), da = l - la, db = l - lb;
    const float cut = tab[0][l];
    const int k = (mode & 2) ? db : da + db;  // log2 of the size of item 2 in cells of the finer level
    const float acc = tab[1][k], can = tab[2][k];
    int X = ((2 * xln_ix(a.x) + 1) << da) - ((2 * xln_ix(b.x) + 1) << db);
    int Y = ((2 * a.y + 1) << da) - ((2 * b.y + 1) << db);
    int Z = ((2 * a.z + 1) << da) - ((2 * b.z + 1) << db);
    if (__ballot(s != 13)) {  // some pair is with a periodic image
        const int sx = (s * 57) >> 9, q = s - 9 * sx, sy = (q * 11) >> 5, sz = q - 3 * sy;
        X -= (int)((unsigned)(sx - 1) << (l + 1));
        Y -= (int)((unsigned)(sy - 1) << (l + 1));
        Z -= (int)((unsigned)(sz - 1) << (l + 1));
    }
    const float half = (float)((1 << da) + (1 << db));
    const float ax = fabsf((float)X), ay = fabsf((float)Y), az = fabsf((float)Z);
    const float gx = fmaxf(ax - half, 0.0f), gy = fmaxf(ay - half, 0.0f), gz = fmaxf(az - half, 0.0f);
    const float sm2 = fmaf(gx, gx, fmaf(gy, gy, gz * gz)), sc2 = fmaf(ax, ax, fmaf(ay, ay, az * az));
    const float fx = ax + half, fy = ay + half, fz = az + half;
    const float far2 = (mode & 1) ? sc2 : fmaf(fx, fx, fmaf(fy, fy, fz * fz));
    const bool in = !(sm2 > cut), whole = !(far2 > cut);
    MacEval r;
    r.code = in ? (whole && sc2 >= acc ? 1 : 2) : 0;
    r.cand = in && whole && sc2 >= can;
    return r;
}

// Pairs awaiting a decision: positions [0, sp) of a stack whose last entries, from `base` up,
// lie in an LDS ring and the earlier ones in the wave's device memory.
constexpr int kStackLds = 1024;  // a step pushes at most 512 entries

// Sinks t = blockIdx.x, blockIdx.x + gridDim.x, ... of one level.  WHOLE: the acceptance
// criterion on whole numbers in FP32.
template <int MODE, bool WHOLE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MODE == kModeLearned ? 3 : 4))) void k_traverse(TravArgs a, MacConst mc)
{
    constexpr int kM2L = MODE == kModeLearned ? kKindOrd : 0;
    __shared__ __align__(16) short mlp_act[MODE == kModeLearned ? 64 * kActRow : 1];
    __shared__ uint32_t cand_q[MODE == kModeLearned ? kCandQ : 1];
    __shared__ uint32_t stk[kStackLds];
    __shared__ ListRing rings[MODE == kModeExport ? 4 : 3];  // M2L, P2P, handed down, candidates
    __shared__ unsigned char ordring[MODE == kModeLearned ? 2 * kChunk : 1];
    __shared__ float tab[WHOLE ? 3 : 1][kMaxLevel + 1];

    const int lane = threadIdx.x;
    const uint64_t lt = (1ull << lane) - 1ull;
    uint32_t *deep = a.stack + (size_t)blockIdx.x * a.stk_cap;  // the stack below `base`
    const int scap = a.stk_cap;
    const int4 *cellc = a.cellc;
    if (WHOLE && lane <= kMaxLevel) {
        tab[0][lane] = mc.cut[lane];
        tab[WHOLE ? 1 : 0][lane] = mc.acc[lane];
        tab[WHOLE ? 2 : 0][lane] = mc.cand[lane];
    }
    __syncthreads();
    unsigned long long visits = 0, nm2l = 0, np2p = 0, most = 0;
    unsigned nord[kOrders] = {0, 0, 0, 0, 0, 0, 0};  // learned: this wave's M2L pairs per order
    int bnext[kKinds], bend[kKinds];
    int *ws = a.wstate + (size_t)blockIdx.x * 2 * kKinds;
#pragma unroll
    for (int k = 0; k < kKinds; ++k) {
        bnext[k] = __builtin_amdgcn_readfirstlane(ws[k]);
        bend[k] = __builtin_amdgcn_readfirstlane(ws[kKinds + k]);
    }
    for (int t = xcd_order(blockIdx.x, gridDim.x); t < a.ln; t += gridDim.x) {
        const int A = a.lbeg + t;
        const int4 ga = cellc[A];
        const int4 ra = reinterpret_cast<const int4 *>(a.cells)[2 * (size_t)A + 1];  // beg, end, parent
        const int parentA = ra.z, nA = ra.y - ra.x;
        const bool leafA = xln_nchild(ga.x) == 0;
        const int lvA = xln_level(ga.x);
        const bool root = lvA == 0;  // a root meets the 27 periodic images of itself
        int ninh = 27, ichunk = 0;
        if (root && nA == 0) ninh = 0;  // empty box of a batch: nothing to do
        if (!root) {
            ninh = __builtin_amdgcn_readfirstlane(a.cnt[2 * a.ncell + parentA]);
            ichunk = __builtin_amdgcn_readfirstlane(a.head[2 * a.ncell + parentA]);
        }
        double mA0 = 0.0;
        if (MODE == kModeLearned) mA0 = a.cf[A].x;
        ListState Lm{-1, -1, 0}, Lp{-1, -1, 0}, Ld{-1, -1, 0}, Lc{-1, -1, 0};
        unsigned oc[kOrders] = {0, 0, 0, 0, 0, 0, 0};  // learned: this sink's M2L pairs per order
        int qhead = 0, qtail = 0;  // learned: queue of candidate pairs awaiting the selector
        bool failed = false;
        // the inherited pairs go onto the stack first, so every step takes a full batch of
        // 64 while that many are pending (opened sources push their children on top)
        if (ninh > scap) {
            if (lane == 0) atomicOr(a.err, 1);
            continue;
        }
        int sp = ninh, base = ninh > kStackLds ? (ninh - kStackLds + 63) & ~63 : 0;
        if (root) {
            if (lane < ninh) stk[lane] = (uint32_t)A << 5 | (uint32_t)lane;
        } else {
            for (int e0 = 0; e0 < ninh; e0 += kChunk) {
                const uint32_t v = a.items[2][(size_t)ichunk * kChunk + lane];
                if (e0 + kChunk < ninh) ichunk = __builtin_amdgcn_readfirstlane(a.next[2][ichunk]);
                if (e0 >= base) stk[(e0 + lane) & (kStackLds - 1)] = v;  // past ninh: free slots
                else deep[e0 + lane] = v;                               // base is a multiple of 64
            }
        }
        lds_order();

        for (;;) {
            // next batch: a flush of the candidate queue (learned: when 64 wait, or when
            // nothing else is left), else up to 64 pairs from the stack
            int kk = 0, fk = 0;
            uint32_t it = 0;
            if (MODE == kModeLearned && qtail - qhead >= 64) {
                fk = 64;
            } else if (sp > 0) {
                kk = sp < 64 ? sp : 64;
                if (sp - kk < base) {  // the LDS part holds less than the batch: fetch half a ring below it
                    __syncthreads();
                    const int nb = base > kStackLds / 2 ? base - kStackLds / 2 : 0;
                    for (int p = nb; p < base; p += 64) stk[(p + lane) & (kStackLds - 1)] = deep[p + lane];
                    base = nb;
                    lds_order();
                }
                sp -= kk;
                it = stk[(sp + lane) & (kStackLds - 1)];
            } else if (MODE == kModeLearned && qtail > qhead) {
                fk = qtail - qhead;
            } else {
                break;
            }
            bool valid, opened;
            int ord;
            int4 gb = make_int4(0, 0, 0, 0);
            if (MODE == kModeLearned && fk > 0) {
                // the selector decides fk queued candidates at once (features, MLP on the
                // matrix cores, order decoding); not accepted means opened
                lds_order();
                valid = lane < fk;
                it = valid ? cand_q[(qhead + lane) & (kCandQ - 1)] : 0u;
                qhead += fk;
                const int B = (int)(it >> 5), s = (int)(it & 31);
                float fv[kFeat];
                for (int q = 0; q < kFeat; ++q) fv[q] = 0.0f;
                if (valid) {
                    gb = cellc[B];
                    PairGeo g = pair_geo(ga, gb, s);
                    pair_features(g, lvA, xln_level(gb.x), a.box, a.rs, a.rcut, mA0, a.cf[B], fv);
                }
                float lg[kCls];
                mlp_logits_wave(a.model->w, fv, mlp_act, lg);
                ord = valid ? decode_order(lg, a.model->safety) : 0;
                opened = ord < 2;
#pragma unroll
                for (int o = 0; o < kOrders; ++o) oc[o] += __popcll(__ballot(valid && ord == o + 2));
            } else {
                visits += kk;
                valid = lane < kk;
                it = valid ? it : (uint32_t)A << 5 | 13u;  // lanes past the batch: the sink itself, not used
                const int B = (int)(it >> 5), s = (int)(it & 31);
                gb = cellc[B];
                MacEval ev{0, false};
                if (WHOLE) ev = mac_whole(ga, lvA, gb, s, mc.mode, tab);
                else if (MODE == kModePlain) ev.code = mac_decide(ga, gb, s, mc);
                else ev = mac_eval(ga, gb, s, mc, a.theta_max2);
                const int d = valid ? ev.code : 0;
                const bool cand = valid && ev.cand;
                if (MODE == kModeExport)
                    emit(a, kKindCand, Lc, rings[MODE == kModeExport ? 3 : 0], nullptr, bnext, bend, cand, it, lt, lane);
                if (MODE == kModeLearned) {
                    // candidates wait in the queue; the rest are pruned (d = 0) or opened
                    const uint64_t cm = __ballot(cand);
                    if (cand) cand_q[(qtail + __popcll(cm & lt)) & (kCandQ - 1)] = it;
                    qtail += __popcll(cm);
                    valid = valid && !cand;
                    ord = 0;
                    opened = d != 0;
                } else {
                    ord = d == 1 ? 2 : 0;
                    opened = d == 2;
                }
            }
            // lists and stack: `ord` >= 2 puts the pair on an M2L list (order ord in learned
            // mode, else plain), `opened` hands it to P2P, to the children of A, or opens
            // the source
            const bool leafB = xln_nchild(gb.x) == 0;
            opened = valid && opened;
            const bool is_p2p = opened && leafA && leafB;
            const bool is_pd = opened && !is_p2p && !leafA && (lvA <= xln_level(gb.x) || leafB);
            const bool open_src = opened && !is_p2p && !is_pd;
            emit<MODE == kModeLearned>(a, kM2L, Lm, rings[0], ordring, bnext, bend, valid && ord >= 2, it, lt, lane,
                                       (unsigned char)ord);
            emit(a, 1, Lp, rings[1], nullptr, bnext, bend, is_p2p, it, lt, lane);
            emit(a, 2, Ld, rings[2], nullptr, bnext, bend, is_pd, it, lt, lane);
            if (__ballot(open_src) == 0) continue;
            const int nch = open_src ? xln_nchild(gb.x) : 0;
            const int incl = wave_incl_sum(nch);
            const int tot = __builtin_amdgcn_readlane(incl, 63);
            if (sp + tot > scap) {
                if (lane == 0) atomicOr(a.err, 1);
                failed = true;
                break;
            }
            if (sp + tot > base + kStackLds) {  // room in the ring: its older half moves out
                for (int p = base; p < base + kStackLds / 2; p += 64) deep[p + lane] = stk[(p + lane) & (kStackLds - 1)];
                base += kStackLds / 2;
                lds_order();
            }
            const int off = sp + incl - nch;
            const uint32_t first = (uint32_t)gb.w << 5 | (it & 31u);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (q < nch) stk[(off + q) & (kStackLds - 1)] = first + ((uint32_t)q << 5);
            sp += tot;
            lds_order();
        }
        if (failed) continue;
        // the open ends of the lists
        lds_order();
        auto close = [&](int k, ListState &L, const ListRing &ring) __attribute__((always_inline)) {
            if (L.tot & (kChunk - 1))
                flush<false>(a, k, L, ring, nullptr, bnext, bend, L.tot & ~(kChunk - 1), L.tot & (kChunk - 1), lane);
            if (lane == 0) {
                a.head[k * a.ncell + A] = L.head;
                a.cnt[k * a.ncell + A] = L.tot;
            }
        };
        if (MODE == kModeLearned) {
            if (Lm.tot & (kChunk - 1))
                flush<true>(a, kM2L, Lm, rings[0], ordring, bnext, bend, Lm.tot & ~(kChunk - 1), Lm.tot & (kChunk - 1), lane);
            if (lane == 0) {
                a.head[kM2L * a.ncell + A] = Lm.head;
                a.cnt[kM2L * a.ncell + A] = Lm.tot;
            }
        } else {
            close(kM2L, Lm, rings[0]);
        }
        close(1, Lp, rings[1]);
        close(2, Ld, rings[2]);
        if (MODE == kModeExport) close(kKindCand, Lc, rings[MODE == kModeExport ? 3 : 0]);
        lds_order();
        nm2l += Lm.tot;
        np2p += Lp.tot;
        if (Lp.tot > 0) {
            const unsigned long long c = (unsigned long long)Lp.tot * ((nA + a.tile - 1) / a.tile);
            most = c > most ? c : most;
        }
        if (MODE == kModeLearned) {
#pragma unroll
            for (int o = 0; o < kOrders; ++o) {
                if (lane == 0) a.ocnt[(size_t)o * a.ncell + A] = (int)oc[o];
                nord[o] += oc[o];
            }
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kKinds; ++k) {
            ws[k] = bnext[k];
            ws[kKinds + k] = bend[k];
        }
        unsigned long long *c = a.slots + (size_t)(blockIdx.x % kTravSlots) * kSlotWords;
        atomicAdd(&c[0], visits);
        atomicAdd(&c[1], nm2l);
        atomicAdd(&c[2], np2p);
        if (MODE == kModeLearned)
            for (int k = 0; k < kOrders; ++k) atomicAdd(&c[3 + k], (unsigned long long)nord[k]);
        if (most > 0) atomicMax(&c[3 + kOrders], most);
    }
}

// Smallest whole s with pass(s), pass monotone and guessed to begin near `guess`; "none" past
// 2^24, which no squared distance that reaches the test exceeds in the whole-number form.
template <class F> static float first_whole(double guess, F pass)
{
    if (!(guess < 16777218.0)) return 3.0e38f;
    double s = ceil(guess);
    s = s > 0.0 ? s : 0.0;
    while (s > 0.0 && pass(s - 1.0)) s -= 1.0;
    while (s < 16777218.0 && !pass(s)) s += 1.0;
    return s > 16777216.0 ? 3.0e38f : (float)s;
}

// Thresholds of the traversal.  The whole-number form needs a squared cutoff below 2^24 at
// the tree's finest level (r_cut below 4096 cell halves there) and a criterion that never
// looks beyond the cutoff (not the conventional one).
static void mac_setup(const fmm_params *P, double theta_max, int nlevel, MacConst &mc)
{
    const double u0 = 0.5 * P->box;
    mc.cut2 = (P->r_cut * P->r_cut) / (u0 * u0);
    mc.theta2 = P->theta * P->theta;
    mc.mode = P->mac_mode;
    mc.whole = !(mc.mode & 4) && nlevel <= kMaxLevel + 1 && ldexp(mc.cut2, 2 * (nlevel - 1)) < 16777216.0;
    const double tm2 = theta_max * theta_max;
    for (int l = 0; l <= kMaxLevel; ++l) {
        const double c = floor(ldexp(mc.cut2, 2 * l)), w = ldexp(4.0, 2 * l);
        mc.cut[l] = c < 16777216.0 ? (float)c : 3.0e38f;
        mc.acc[l] = first_whole(w / mc.theta2, [&](double s) { return w <= mc.theta2 * s; });
        mc.cand[l] = tm2 > 0.0 ? first_whole(w / tm2, [&](double s) { return w / s <= tm2; }) : 3.0e38f;
    }
}

// Waves of one traversal kernel that fit on the device at once.  Sinks are dealt to the
// waves statically, so the grid is never larger than this: a second partial round of
// waves would only lengthen the tail of each level.
template <int MODE> static int resident_waves()
{
    static int cached = 0;
    if (cached == 0) {
        int dev = 0, ncu = 0, per = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_traverse<MODE, true>, 64, 0) != hipSuccess)
            return 4096;
        cached = (ncu > 0 ? ncu : 1) * (per > 0 ? per : 1);
    }
    return cached;
}

static int resident_waves(int mode)
{
    if (mode == kModePlain) return resident_waves<kModePlain>();
    if (mode == kModeExport) return resident_waves<kModeExport>();
    return resident_waves<kModeLearned>();
}

// The traversal's 16-byte view of each cell, packed: the random cell reads of the traversal
// then touch half as many cache lines (8 sibling cells per 128-byte line).
__global__ void k_pack_cells(const Cell *__restrict__ cells, int ncell, int4 *__restrict__ out)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < ncell) out[c] = reinterpret_cast<const int4 *>(cells)[2 * (size_t)c];
}

// Per-cell part of the selector's features, from the scaled multipoles (stride `stride`).
template <class T>
__global__ void k_cell_features(const T *__restrict__ M, int stride, int ncell, float4 *__restrict__ cf)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < ncell) cf[c] = cell_features<T>(M + (size_t)c * stride);
}

// Wave w starts with chunks [w kChunkBlock, (w+1) kChunkBlock) of every list kind, and
// the counters start past those blocks: no wave needs an atomic for its first block.
__global__ void k_wstate_init(int *ws, int nw, int *pool)
{
    int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w < nw)
        for (int k = 0; k < kKinds; ++k) {
            ws[(size_t)w * 2 * kKinds + k] = w * kChunkBlock;
            ws[(size_t)w * 2 * kKinds + kKinds + k] = (w + 1) * kChunkBlock;
        }
    if (w == 0)
        for (int k = 0; k < kKinds; ++k) pool[k * kPoolStride] = nw * kChunkBlock;
}

static int ensure_pools(fmm_tree *t, const int *want)
{
    for (int k = 0; k < kKinds; ++k) {
        if (want[k] <= t->lcap[k]) continue;
        int cap = want[k] + want[k] / 4 + 64;
        if (int rc = grow(t->litems[k], (size_t)(cap + 1) * kChunk * 4) | grow(t->lnext[k], (size_t)(cap + 1) * 4))
            return rc;
        if (k == kKindOrd)
            if (int rc = grow(t->lord, (size_t)(cap + 1) * kChunk)) return rc;
        t->lcap[k] = cap;
    }
    return 0;
}

// mode: kModePlain / kModeExport / kModeLearned.  For the last two, theta_max bounds the
// candidates, M/mstride/mprec give the multipoles used by the features, model the
// selector (learned only).
int traverse_mode(fmm_tree *t, const fmm_params *P, int mode, double theta_max, const void *M, int mstride,
                  int mprec, const MacModel *model, hipStream_t st, const TravHook *hook)
{
    MacConst mc;
    mac_setup(P, theta_max, t->nlevel, mc);
    const int ncell = t->ncell;
    // lcnt: kKinds list sizes, then the learned selector's per-order counts
    const size_t ncnt = (size_t)(kKinds + (mode == kModeLearned ? kOrders : 0)) * ncell;
    int rc = grow(t->lhead, (size_t)kKinds * ncell * 4) | grow(t->lcnt, (size_t)(kKinds + kOrders) * ncell * 4) |
             grow(t->counters, kCounterBytes);
    if (rc) return rc;
    // list kinds written in this mode get room for their expected size plus the partly
    // used chunk block each wave may hold at the end
    int want[kKinds];
    const int slack = resident_waves(mode) * kChunkBlock + 64;
    for (int k = 0; k < kKinds; ++k) want[k] = 0;
    want[1] = slack + 8 * t->nleaf;
    want[2] = slack + 2 * ncell;
    if (mode == kModeLearned) {
        want[kKindOrd] = slack + 4 * ncell;
    } else {
        want[0] = slack + 2 * ncell;
        if (mode == kModeExport) want[kKindCand] = slack + 2 * ncell;
    }
    if ((rc = ensure_pools(t, want))) return rc;
    if ((rc = grow(t->cellc, (size_t)ncell * sizeof(int4)))) return rc;
    k_pack_cells<<<(ncell + 255) / 256, 256, 0, st>>>(ptr<Cell>(t->cells), ncell, ptr<int4>(t->cellc));
    if (mode == kModeLearned) {
        if (!M || mstride < 20) return set_error(FMM_ERR_ARG, "learned traversal: multipoles of order >= 3 needed");
        if ((rc = grow(t->cfeat, (size_t)ncell * sizeof(float4)))) return rc;
        if (mprec)
            k_cell_features<float><<<(ncell + 63) / 64, 64, 0, st>>>(static_cast<const float *>(M), mstride, ncell,
                                                                    ptr<float4>(t->cfeat));
        else
            k_cell_features<double><<<(ncell + 63) / 64, 64, 0, st>>>(static_cast<const double *>(M), mstride, ncell,
                                                                     ptr<float4>(t->cfeat));
    }
    for (int attempt = 0; attempt < 4; ++attempt) {
        int nw = 1;
        for (int l = 0; l < t->nlevel; ++l) {
            int ln = t->lvl_beg[l + 1] - t->lvl_beg[l];
            nw = ln > nw ? ln : nw;
        }
        const int cap = resident_waves(mode);
        nw = nw < cap ? nw : cap;
        if ((rc = grow(t->tstack, (size_t)nw * t->stk_cap * 4))) return rc;
        if ((rc = grow(t->wstate, (size_t)nw * 2 * kKinds * sizeof(int)))) return rc;
        unsigned char *cb = ptr<unsigned char>(t->counters);
        if ((rc = zero_async(cb, kCounterBytes, st))) return rc;  // a kernel: also valid inside a recorded graph
        k_wstate_init<<<(nw + 255) / 256, 256, 0, st>>>(ptr<int>(t->wstate), nw,
                                                        reinterpret_cast<int *>(cb + kPoolByte));
        if ((rc = zero_async(t->lcnt.p, ncnt * 4, st))) return rc;
        TravArgs a;
        a.cells = ptr<Cell>(t->cells);
        a.ncell = ncell;
        for (int k = 0; k < kKinds; ++k) {
            a.items[k] = ptr<uint32_t>(t->litems[k]);
            a.next[k] = ptr<int>(t->lnext[k]);
            a.cap[k] = t->lcap[k];
        }
        a.tile = p2p_tile(P);
        a.slots = reinterpret_cast<unsigned long long *>(cb + kTravByte);
        a.pool = reinterpret_cast<int *>(cb + kPoolByte);
        a.wstate = ptr<int>(t->wstate);
        a.err = reinterpret_cast<int *>(cb + kErrByte);
        a.head = ptr<int>(t->lhead);
        a.cnt = ptr<int>(t->lcnt);
        a.ord = ptr<unsigned char>(t->lord);
        a.ocnt = ptr<int>(t->lcnt) + (size_t)kKinds * ncell;
        a.stack = ptr<uint32_t>(t->tstack);
        a.stk_cap = t->stk_cap;
        a.theta_max2 = theta_max * theta_max;
        a.box = P->box;
        a.rs = P->r_s;
        a.rcut = P->r_cut;
        a.cf = ptr<float4>(t->cfeat);
        a.model = model;
        a.cellc = ptr<int4>(t->cellc);
        for (int l = 0; l < t->nlevel; ++l) {
            a.lbeg = t->lvl_beg[l];
            a.ln = t->lvl_beg[l + 1] - a.lbeg;
            int g = a.ln < nw ? a.ln : nw;
            if (mc.whole) {
                if (mode == kModePlain) k_traverse<kModePlain, true><<<g, 64, 0, st>>>(a, mc);
                else if (mode == kModeExport) k_traverse<kModeExport, true><<<g, 64, 0, st>>>(a, mc);
                else k_traverse<kModeLearned, true><<<g, 64, 0, st>>>(a, mc);
            } else {
                if (mode == kModePlain) k_traverse<kModePlain, false><<<g, 64, 0, st>>>(a, mc);
                else if (mode == kModeExport) k_traverse<kModeExport, false><<<g, 64, 0, st>>>(a, mc);
                else k_traverse<kModeLearned, false><<<g, 64, 0, st>>>(a, mc);
            }
            if (hook)
                if ((rc = hook->level(hook->ctx, l, st))) return rc;
        }
        if ((rc = hip_check(hipGetLastError(), "traversal"))) return rc;
        // Being recorded: the tree and parameters are those of the evaluation just run, whose
        // pools and stacks fitted; the lists, their sizes and every wave's use of pool blocks
        // and stack (sinks are dealt statically) repeat exactly, so no readback is needed.
        if (t->capturing) return 0;
        if ((rc = hip_check(hipMemcpyAsync(t->host, cb, kP2PByte, hipMemcpyDeviceToHost, st), "counters")))
            return rc;
        if ((rc = hip_check(hipStreamSynchronize(st), "traversal sync"))) return rc;
        unsigned long long sum[3 + kOrders] = {0}, most = 0;
        int pools[kKinds], err;
        for (int s = 0; s < kTravSlots; ++s) {
            unsigned long long c[4 + kOrders];
            memcpy(c, (char *)t->host + kTravByte + (size_t)s * kSlotWords * 8, sizeof(c));
            for (int k = 0; k < 3 + kOrders; ++k) sum[k] += c[k];
            most = c[3 + kOrders] > most ? c[3 + kOrders] : most;
        }
        for (int k = 0; k < kKinds; ++k)  // kinds this mode does not write keep their size
            pools[k] = want[k] ? t->host[kPoolByte / 4 + k * kPoolStride] : 0;
        memcpy(&err, (char *)t->host + kErrByte, 4);
        if (err == 0) {
            for (int k = 0; k < kOrders; ++k) t->stats.n_m2l_by_order[k] = mode == kModeLearned ? (int64_t)sum[3 + k] : 0;
            t->n_visit = (int64_t)sum[0];
            t->n_m2l = (int64_t)sum[1];
            t->n_p2p = (int64_t)sum[2];
            t->p2p_max_cost = (int64_t)most;
            t->trav_mode = mode;
            return 0;
        }
        // what the hook launched read the counters the rerun clears: let it end first
        if (hook && hook->side)
            if ((rc = hip_check(hipStreamSynchronize(hook->side), "traversal side stream"))) return rc;
        if (err & 1) t->stk_cap *= 4;  // a wave's stack overflowed: larger stacks, rerun
        if (err & 2)
            if ((rc = ensure_pools(t, pools))) return rc;
    }
    return set_error(FMM_ERR_NOMEM, "traversal did not fit after resizing");
}

int traverse(fmm_tree *t, const fmm_params *P, hipStream_t st, const TravHook *hook)
{
    return traverse_mode(t, P, kModePlain, 0.0, nullptr, 0, 0, nullptr, st, hook);
}

}  // namespace hfmm
