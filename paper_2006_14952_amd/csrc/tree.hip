// Octree construction (the particle packs of Sec. 2.1, built as a Morton octree):
// wrap + 63-bit Morton keys, LSD radix sort (8-bit digits, stable), the leaf depth of each
// particle, SoA gather, and every level's cells at once from the sorted keys.
#include <math.h>

#include "state.h"

namespace hfmm {

// ---------------------------------------------------------------------------
// keys

__device__ inline uint64_t spread3(uint32_t v)  // 21 bits -> every third bit
{
    uint64_t x = v & 0x1fffff;
    x = (x | x << 32) & 0x1f00000000ffffULL;
    x = (x | x << 16) & 0x1f0000ff0000ffULL;
    x = (x | x << 8) & 0x100f00f00f00f00fULL;
    x = (x | x << 4) & 0x10c30c30c30c30c3ULL;
    x = (x | x << 2) & 0x1249249249249249ULL;
    return x;
}

// Periodic wrap into [0, box) and the integer coordinate floor(x / box * 2^21).  The
// expression order (no contraction) fixes the rounding so that every implementation
// of the method assigns a particle to the same cube.
__device__ inline double wrap_coord(double x, double box)
{
#pragma clang fp contract(off)
    double v = x - box * floor(x / box);
    return v >= box ? 0.0 : v;
}

__device__ inline uint32_t grid_coord(double v, double box)
{
#pragma clang fp contract(off)
    double g = floor(v / box * 2097152.0);
    int c = (int)g;
    c = c < 0 ? 0 : c;
    c = c > 2097151 ? 2097151 : c;
    return (uint32_t)c;
}

__global__ void k_keys(const double *__restrict__ pos, int n, double box, uint64_t *__restrict__ keys,
                       uint32_t *__restrict__ idx, int *__restrict__ bad)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double x = pos[3 * (size_t)i], y = pos[3 * (size_t)i + 1], z = pos[3 * (size_t)i + 2];
    if (!isfinite(x) || !isfinite(y) || !isfinite(z)) {
        *bad = 1;
        x = y = z = 0.0;
    }
    uint32_t gx = grid_coord(wrap_coord(x, box), box), gy = grid_coord(wrap_coord(y, box), box),
             gz = grid_coord(wrap_coord(z, box), box);
    keys[i] = spread3(gx) << 2 | spread3(gy) << 1 | spread3(gz);
    idx[i] = (uint32_t)i;
}

// ---------------------------------------------------------------------------
// LSD radix sort, 8-bit digits.  A tile of 256 ROUNDS keys per 256-thread block; each wave
// handles 64 ROUNDS consecutive keys in rounds of 64, ranking equal digits inside a
// round with ballots, so the scatter is stable.

constexpr int kRsThreads = 256;

// Box of original particle index v: the largest b with off[b] <= v (empty boxes skipped).
__device__ inline int box_of(const int *off, int nbox, uint32_t v)
{
    int lo = 0, hi = nbox - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= (int)v) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Radix digit of an element: 8 bits of the Morton key, or (for the passes that group the
// boxes of a batch) 8 bits of the box of its original index.
__device__ inline int rs_digit(uint64_t key, uint32_t val, int shift, const int *boxoff, int nbox)
{
    if (boxoff) return (box_of(boxoff, nbox, val) >> shift) & 0xff;
    return (int)((key >> shift) & 0xff);
}

// Digit counts of each tile: hist[digit][tile], or hist[tile][digit] (OWN, below).
template <int ROUNDS, bool OWN>
__global__ __launch_bounds__(kRsThreads) void k_rs_hist(const uint64_t *__restrict__ keys,
                                                        const uint32_t *__restrict__ vals, int n, int shift,
                                                        const int *__restrict__ boxoff, int nbox, int nblocks,
                                                        int *__restrict__ hist)
{
    __shared__ int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    int base = blockIdx.x * kRsThreads * ROUNDS;
    for (int k = 0; k < ROUNDS; ++k) {
        int i = base + k * kRsThreads + threadIdx.x;
        if (i < n) atomicAdd(&h[rs_digit(keys[i], vals[i], shift, boxoff, nbox)], 1);
    }
    __syncthreads();
    if constexpr (OWN) hist[blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
    else hist[threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// Scatter of one tile: the keys are ranked by digit in registers (ballots, as before),
// placed in LDS in the tile's digit order, and written from there by consecutive threads, so
// each digit's run of the tile goes out as consecutive addresses (whole cache lines) rather
// than as one scattered 8-byte store per key.  offs: the scanned counts; or (OWN, few tiles) the
// counts, from which every tile adds up its own places, instead of one to three launches of a scan.
template <int ROUNDS, bool OWN>
__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(const uint64_t *__restrict__ kin,
                                                           const uint32_t *__restrict__ vin, uint64_t *__restrict__ kout,
                                                           uint32_t *__restrict__ vout, int n, int shift,
                                                           const int *__restrict__ boxoff, int nbox, int nblocks,
                                                           const int *__restrict__ offs)
{
    __shared__ int cnt[4][256];
    __shared__ int boff[256];
    __shared__ int dstart[256];  // first slot of each digit in the tile ordered by digit
    __shared__ int wsum[4];
    constexpr int kRsRounds = ROUNDS, kRsTile = kRsThreads * ROUNDS;
    __shared__ uint64_t skey[kRsTile];
    __shared__ uint32_t sval[kRsTile];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k = threadIdx.x; k < 4 * 256; k += kRsThreads) (&cnt[0][0])[k] = 0;
    if constexpr (OWN) {
        int before = 0, total = 0;
#pragma unroll 16
        for (int b = 0; b < nblocks; ++b) {
            const int c = offs[b * 256 + threadIdx.x];
            total += c;
            before += b < (int)blockIdx.x ? c : 0;
        }
        const int incl = wave_incl_sum(total);
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        for (int q = 0; q < w; ++q) before += wsum[q];
        boff[threadIdx.x] = before + incl - total;
    } else {
        boff[threadIdx.x] = offs[threadIdx.x * nblocks + blockIdx.x];
    }
    __syncthreads();
    const uint64_t lt = (1ull << lane) - 1ull;
    const int base = blockIdx.x * kRsTile + w * (kRsTile / 4);
    uint64_t key[kRsRounds];
    uint32_t val[kRsRounds];
    int pos[kRsRounds];
#pragma unroll
    for (int r = 0; r < kRsRounds; ++r) {
        int i = base + r * 64 + lane;
        bool ok = i < n;
        key[r] = ok ? kin[i] : 0;
        val[r] = ok ? vin[i] : 0;
        int d = rs_digit(key[r], val[r], shift, boxoff, nbox);
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uint64_t m = __ballot((d >> b) & 1);
            peers &= ((d >> b) & 1) ? m : ~m;
        }
        int old = cnt[w][d];
        int rank = __popcll(peers & lt);
        if (ok && rank == 0) cnt[w][d] = old + __popcll(peers);
        pos[r] = ok ? old + rank : -1;
    }
    __syncthreads();
    {  // per-digit prefix over the four waves, then over the digits (a block-wide scan)
        const int d = threadIdx.x;
        int run = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int c = cnt[q][d];
            cnt[q][d] = run;
            run += c;
        }
        const int incl = wave_incl_sum(run);
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        int add = 0;
        for (int q = 0; q < w; ++q) add += wsum[q];
        dstart[d] = add + incl - run;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRsRounds; ++r) {
        if (pos[r] < 0) continue;
        const int d = rs_digit(key[r], val[r], shift, boxoff, nbox);
        const int l = dstart[d] + cnt[w][d] + pos[r];
        skey[l] = key[r];
        sval[l] = val[r];
    }
    __syncthreads();
    const int ntile = min(kRsTile, n - blockIdx.x * kRsTile);
    for (int j = threadIdx.x; j < ntile; j += kRsThreads) {
        const uint64_t k = skey[j];
        const uint32_t v = sval[j];
        const int d = rs_digit(k, v, shift, boxoff, nbox);
        const int o = boff[d] + j - dstart[d];
        kout[o] = k;
        vout[o] = v;
    }
}

// All passes of a small sort in one workgroup: the particles stay in registers, ROUNDS to a
// thread, and change places through LDS; ranks as in k_rs_scatter, over sixteen waves.  Bound by
// the LDS chains of a pass and its five barriers.
template <int ROUNDS>
__global__ __launch_bounds__(1024) void k_rs_small(uint64_t *__restrict__ keys, uint32_t *__restrict__ vals, int n,
                                                   int first_digit, int npass, const int *__restrict__ boxoff, int nbox)
{
    __shared__ int cnt[16][256];
    __shared__ int dstart[256], wsum[4];
    __shared__ uint64_t skey[1024 * ROUNDS];
    __shared__ uint32_t sval[1024 * ROUNDS];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, base = w * 64 * ROUNDS + lane;
    const uint64_t lt = (1ull << lane) - 1ull;
    uint64_t key[ROUNDS];
    uint32_t val[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int i = base + 64 * r;
        key[r] = i < n ? keys[i] : 0;
        val[r] = i < n ? vals[i] : 0;
    }
    for (int pass = first_digit; pass < npass; ++pass) {
        const int shift = pass >= 8 ? 8 * (pass - 8) : 8 * pass;
        const int *bo = pass >= 8 ? boxoff : nullptr;
        for (int k = threadIdx.x; k < 16 * 256; k += 1024) (&cnt[0][0])[k] = 0;
        __syncthreads();
        int pos[ROUNDS], dig[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const bool ok = base + 64 * r < n;
            const int d = rs_digit(key[r], val[r], shift, bo, nbox);
            uint64_t peers = __ballot(ok);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint64_t m = __ballot((d >> b) & 1);
                peers &= ((d >> b) & 1) ? m : ~m;
            }
            const int old = cnt[w][d], rank = __popcll(peers & lt);
            if (ok && rank == 0) cnt[w][d] = old + __popcll(peers);
            dig[r] = d;
            pos[r] = ok ? old + rank : -1;
        }
        __syncthreads();
        int run = 0, incl = 0;
        if (threadIdx.x < 256) {  // per-digit prefix over the waves, then over the digits
            int c[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) c[q] = cnt[q][threadIdx.x];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                cnt[q][threadIdx.x] = run;
                run += c[q];
            }
            incl = wave_incl_sum(run);
            if (lane == 63) wsum[w] = incl;
        }
        __syncthreads();
        if (threadIdx.x < 256) {
            int add = incl - run;
            for (int q = 0; q < w; ++q) add += wsum[q];
            dstart[threadIdx.x] = add;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (pos[r] < 0) continue;
            const int l = dstart[dig[r]] + cnt[w][dig[r]] + pos[r];
            skey[l] = key[r];
            sval[l] = val[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            key[r] = skey[base + 64 * r];
            val[r] = sval[base + 64 * r];
        }
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int i = base + 64 * r;
        if (i < n) {
            keys[i] = key[r];
            vals[i] = val[r];
        }
    }
}

struct RsArgs {
    DevBuf *keys, *idx;
    int n, nbox, first_digit, npass;
    const int *boxoff;
};

template <int ROUNDS, bool OWN>
static int radix_passes(const RsArgs &a, DevBuf &tmp, DevBuf &scan_tmp, int &sorted, hipStream_t st)
{
    constexpr int kRsTile = kRsThreads * ROUNDS;
    const int nb = (a.n + kRsTile - 1) / kRsTile;
    if (int rc = grow(tmp, (size_t)256 * nb * 2 * sizeof(int))) return rc;
    int *hist = ptr<int>(tmp), *offs = OWN ? hist : hist + 256 * nb;
    int cur = sorted;
    for (int pass = a.first_digit; pass < a.npass; ++pass) {
        const int shift = pass >= 8 ? 8 * (pass - 8) : 8 * pass;
        const int *bo = pass >= 8 ? a.boxoff : nullptr;
        const uint64_t *kin = ptr<uint64_t>(a.keys[cur]);
        const uint32_t *vin = ptr<uint32_t>(a.idx[cur]);
        k_rs_hist<ROUNDS, OWN><<<nb, kRsThreads, 0, st>>>(kin, vin, a.n, shift, bo, a.nbox, nb, hist);
        if constexpr (!OWN)
            if (int rc = scan_exclusive(hist, offs, 256 * nb, nullptr, st, scan_tmp)) return rc;
        k_rs_scatter<ROUNDS, OWN><<<nb, kRsThreads, 0, st>>>(kin, vin, ptr<uint64_t>(a.keys[cur ^ 1]),
                                                             ptr<uint32_t>(a.idx[cur ^ 1]), a.n, shift, bo, a.nbox, nb,
                                                             offs);
        cur ^= 1;
    }
    sorted = cur;
    return hip_check(hipGetLastError(), "radix sort");
}

// Passes over the Morton key's digits first_digit .. 7, then (batches) 1 or 2 passes over
// the box index, so the order is by box, then by key; stable throughout.  Sorts the buffer
// pair `sorted` of keys and idx (0 after k_keys) and sets it to the pair with the result.
//
// Three forms, by the time of a whole tree build (us, clustered boxes):
//   n                                   4,096  8,192  16,384  65,536  131,072  524,288  1,048,576  2,097,152
//   one workgroup                         124    148
//   tiles of 1,024 that add up places     161    179     168     175      192      288        500      1,255
//   tiles of 2,048, the same              179    191     194     196      205      262        349        610
//   tiles of 4,096 and a scan             214    249     255     295      305      332        364        453
// Small sorts are bound by the launches of six passes, in sequence some 20 us a pass with the
// scan; large ones by memory, and the tiles' own sums grow with the square of their number.
static int radix_sort(DevBuf (&keys)[2], DevBuf (&idx)[2], DevBuf &tmp, DevBuf &scan_tmp, int &sorted, int n,
                      const int *boxoff, int nbox, int first_digit, hipStream_t st)
{
    const RsArgs a{keys, idx, n, nbox, first_digit, 8 + (nbox > 1) + (nbox > 256), boxoff};
    auto small = [&](auto kernel) {
        kernel<<<1, 1024, 0, st>>>(ptr<uint64_t>(keys[sorted]), ptr<uint32_t>(idx[sorted]), n, first_digit, a.npass,
                                   boxoff, nbox);
        return hip_check(hipGetLastError(), "radix sort");
    };
    if (n <= 1 << 10) return small(k_rs_small<1>);
    if (n <= 1 << 11) return small(k_rs_small<2>);
    if (n <= 1 << 12) return small(k_rs_small<4>);
    if (n <= 1 << 13) return small(k_rs_small<8>);
    if (n <= 1 << 17) return radix_passes<4, true>(a, tmp, scan_tmp, sorted, st);
    if (n <= 1 << 20) return radix_passes<8, true>(a, tmp, scan_tmp, sorted, st);
    return radix_passes<16, false>(a, tmp, scan_tmp, sorted, st);
}

// ---------------------------------------------------------------------------
// The cells from the sorted keys, without a loop over the levels.
//
// Particle i begins a cell at every level from d_i, the first level at which its key differs
// from its predecessor's (0 for the first particle of a box), down to D_i, the level of the
// leaf it lies in: the cells are the pairs (i, l) with d_i <= l <= D_i.  A level-l cell splits
// if it holds more than n_crit particles, i.e. if n_crit + 1 consecutive particles share it;
// so D_i is one more than the deepest level shared by any such window over i:
//   D_i = max over j in [i - n_crit, i] of e_j,  e_j = 1 + level shared by keys j and j + n_crit
// (0 where that window leaves the box).  Counting the cells and leaves that begin in each
// tile of particles, level by level, and one scan over (level, tile) number them breadth
// first; a second pass over the particles writes them.  Bound by memory latency on small
// boxes, by the key reads on large ones: seven to nine launches after the sort, where seven
// per level made about 110.

__device__ inline uint32_t compact3(uint64_t x)  // every third bit -> 21 bits
{
    x &= 0x1249249249249249ULL;
    x = (x | x >> 2) & 0x10c30c30c30c30c3ULL;
    x = (x | x >> 4) & 0x100f00f00f00f00fULL;
    x = (x | x >> 8) & 0x1f0000ff0000ffULL;
    x = (x | x >> 16) & 0x1f00000000ffffULL;
    x = (x | x >> 32) & 0x1fffff;
    return (uint32_t)x;
}

// What the tree passes read.  lmax: the deepest level the keys' order is exact to (a partial
// sort's 15, or 21).
struct TreeIn {
    const uint64_t *keys;
    const int *boxoff;
    int n, nbox, ncrit, lmax;
};

// Levels shared by two keys, at most lmax.
__device__ __forceinline__ int shared_levels(uint64_t a, uint64_t b, int lmax)
{
    const uint64_t x = a ^ b;
    const int c = x ? (__clzll((long long)x) - 1) / 3 : kMaxLevel;
    return c < lmax ? c : lmax;
}

__device__ __forceinline__ int tree_box(const TreeIn &t, int i) { return t.nbox > 1 ? box_of(t.boxoff, t.nbox, i) : 0; }
__device__ __forceinline__ int box_end(const TreeIn &t, int b) { return t.nbox > 1 ? t.boxoff[b + 1] : t.n; }

// e_j (0 where j or the window's end lies outside)
__device__ __forceinline__ int window_level(const TreeIn &t, int64_t j)
{
    if (j < 0 || j + t.ncrit >= t.n) return 0;
    const int a = (int)j, b = a + t.ncrit;
    if (t.nbox > 1 && b >= t.boxoff[box_of(t.boxoff, t.nbox, a) + 1]) return 0;
    return 1 + shared_levels(t.keys[a], t.keys[b], t.lmax);
}

// d_i; past lmax (no cell begins) if the particle shares level lmax with its predecessor
__device__ __forceinline__ int first_level(const TreeIn &t, int i, int b, uint64_t key)
{
    if (i == (t.nbox > 1 ? t.boxoff[b] : 0)) return 0;
    return 1 + shared_levels(key, t.keys[i - 1], t.lmax);
}

// Tiles of 256 ITEMS particles, runs of 64 of them to a wave.
constexpr int kTreeThreads = 256;
constexpr int kTreeWin = 512;                // widest window (n_crit) whose maximum is taken in LDS

// Widest windows: e_j for j >= -n_crit in bytes, then maxima over 2, 4, ... of them.
__global__ void k_window_levels(TreeIn t, unsigned char *__restrict__ e, int len)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < len) e[q] = (unsigned char)window_level(t, (int64_t)q - t.ncrit);
}

__global__ void k_window_max(const unsigned char *__restrict__ in, unsigned char *__restrict__ out, int len, int step)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= len) return;
    const unsigned char a = in[q], b = (int64_t)q + step < len ? in[q + step] : 0;
    out[q] = a > b ? a : b;
}

// Depths D_i and, per tile and level, the cells and the leaves that begin there:
// count[(l - 1) nblk + tile] and count[(21 + l - 1) nblk + tile] for l = 1 .. 21.
// win: maxima over 2^wexp entries of the window array (wide windows), else nullptr.
template <int ITEMS>
__global__ __launch_bounds__(kTreeThreads) void k_depth(TreeIn t, const unsigned char *__restrict__ win, int wexp,
                                                        unsigned char *__restrict__ depth, int nblk,
                                                        int *__restrict__ count, int *__restrict__ deep)
{
    constexpr int kTreeTile = kTreeThreads * ITEMS;
    __shared__ unsigned char m[2][kTreeTile + kTreeWin];
    __shared__ int cnt[2][kMaxLevel];
    const int lane = threadIdx.x & 63;
    const int base = blockIdx.x * kTreeTile;
    if (threadIdx.x < 2 * kMaxLevel) (&cnt[0][0])[threadIdx.x] = 0;
    int cur = 0;
    if (!win && t.ncrit < t.n) {
        const int len = kTreeTile + t.ncrit;
        for (int q = threadIdx.x; q < len; q += kTreeThreads)
            m[0][q] = (unsigned char)window_level(t, (int64_t)base - t.ncrit + q);
        __syncthreads();
        for (int k = 0; k < wexp; ++k) {
            for (int q = threadIdx.x; q < len; q += kTreeThreads) {
                const int o = q + (1 << k);
                m[cur ^ 1][q] = max(m[cur][q], o < len ? m[cur][o] : (unsigned char)0);
            }
            __syncthreads();
            cur ^= 1;
        }
    } else {
        __syncthreads();
    }
    bool isdeep = false;
    for (int k = 0; k < ITEMS; ++k) {
        const int p = k * kTreeThreads + threadIdx.x, i = base + p;
        const bool valid = i < t.n;
        int d = kMaxLevel + 1, D = 0;
        if (valid) {
            if (t.ncrit < t.n) {  // the window starts i - n_crit .. i, as two overlapping runs of 2^wexp
                const int64_t lo = win ? (int64_t)i : (int64_t)p, hi = lo + t.ncrit + 1 - (1 << wexp);
                D = win ? max(win[lo], win[hi]) : max(m[cur][lo], m[cur][hi]);
            }
            isdeep |= D > t.lmax;
            D = D < kMaxLevel ? D : kMaxLevel;
            depth[i] = (unsigned char)D;
            const int b = tree_box(t, i);
            d = first_level(t, i, b, t.keys[i]);
        }
        const bool starts = valid && d <= D;
        uint64_t left = __ballot(starts);
        int lo = starts ? d : kMaxLevel + 1, hi = starts ? D : 0;
        if (left) {
            for (int o = 32; o > 0; o >>= 1) {
                lo = min(lo, __shfl_xor(lo, o, 64));
                hi = max(hi, __shfl_xor(hi, o, 64));
            }
            for (int l = lo > 1 ? lo : 1; l <= hi; ++l) {
                const uint64_t mc = __ballot(starts && d <= l && l <= D), ml = __ballot(starts && D == l);
                if (lane == 0) {
                    if (mc) atomicAdd(&cnt[0][l - 1], __popcll(mc));
                    if (ml) atomicAdd(&cnt[1][l - 1], __popcll(ml));
                }
            }
        }
    }
    if (isdeep && t.lmax < kMaxLevel) *deep = 1;
    __syncthreads();
    if (threadIdx.x < 2 * kMaxLevel)
        count[(size_t)threadIdx.x * nblk + blockIdx.x] = (&cnt[0][0])[threadIdx.x];
}

// One workgroup: the roots (level 0, one per box, empty boxes too).  out: their cells, and
// their places among the leaves and the cells with children; or (cells nullptr) what the host
// sizes the tree by: the roots' leaf count, the scan of count at the first tile of every level,
// starts[0 .. 41], and its total, starts[42].
__global__ __launch_bounds__(1024) void k_roots(const int *__restrict__ boxoff, int nbox, int ncrit,
                                                Cell *__restrict__ cells, int *__restrict__ leaves,
                                                int *__restrict__ inner, int *__restrict__ nleaf0,
                                                const int *__restrict__ count, const int *__restrict__ scan, int nblk,
                                                int *__restrict__ starts)
{
    constexpr int kRows = 2 * kMaxLevel;
    if (starts && threadIdx.x <= kRows) {
        const size_t end = (size_t)kRows * nblk - 1, at = (size_t)threadIdx.x * nblk;
        starts[threadIdx.x] = threadIdx.x < kRows ? scan[at] : scan[end] + count[end];
    }
    __shared__ int wsum[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int before = 0;
    for (int b0 = 0; b0 < nbox; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        const int beg = b < nbox ? boxoff[b] : 0, end = b < nbox ? boxoff[b + 1] : 0;
        const bool leaf = b < nbox && end - beg <= ncrit;
        const uint64_t m = __ballot(leaf);
        if (lane == 0) wsum[w] = __popcll(m);
        __syncthreads();
        int rank = before + __popcll(m & ((1ull << lane) - 1ull)), tot = 0;
        for (int q = 0; q < 16; ++q) {
            if (q < w) rank += wsum[q];
            tot += wsum[q];
        }
        if (cells && b < nbox) {
            Cell c;
            c.xln = pack_xln(0, 0, 0);
            c.iy = c.iz = 0;
            c.pad = 0;
            c.beg = beg;
            c.end = end;
            c.child = -1;
            c.parent = -1;
            cells[b] = c;
            if (leaves) {
                if (leaf) leaves[rank] = b;
                else inner[b - rank] = b;
            }
        }
        before += tot;
        __syncthreads();
    }
    if (nleaf0 && threadIdx.x == 0) *nleaf0 = before;
}

// The cells of levels 1 .. 21 (all but the child counts), the leaf and inner-cell lists and
// the leaf of each particle.  Each wave takes runs of 64 particles; a level's cells that begin
// in the run are numbered by ballots.  The cells that reach past their run, at most one a level,
// all hold the run's last particle: their ends are searched for first, a thread per run and
// level.  Searched for level by level where the cells are written, the dependent key reads took
// most of the pass: 262k box 40 -> 26 us, 2M box 62 -> 43, 16.7M box 312 -> 246.
template <int ITEMS>
__global__ __launch_bounds__(kTreeThreads) void k_cells(TreeIn t, const unsigned char *__restrict__ depth, int nblk,
                                                        const int *__restrict__ scan, int nleaf0,
                                                        Cell *__restrict__ cells, int *__restrict__ leaves,
                                                        int *__restrict__ inner, int *__restrict__ leaf_of)
{
    constexpr int kTreeTile = kTreeThreads * ITEMS, kTreeChunks = kTreeTile / 64;
    __shared__ int cc[kTreeChunks][kMaxLevel + 1], cl[kTreeChunks][kMaxLevel + 1];
    __shared__ int ends[kTreeChunks][kMaxLevel + 1], open[kTreeChunks][2];  // open: levels to search, [0] .. [1]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = (1ull << lane) - 1ull, le = lt | 1ull << lane;
    const int base = blockIdx.x * kTreeTile;
    for (int q = threadIdx.x; q < kTreeChunks * (kMaxLevel + 1); q += kTreeThreads) {
        (&cc[0][0])[q] = 0;
        (&cl[0][0])[q] = 0;
    }
    __syncthreads();
    uint64_t key[ITEMS];
    int box[ITEMS], d[ITEMS], D[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = base + k * kTreeThreads + threadIdx.x, ch = k * (kTreeThreads / 64) + w;
        key[k] = 0;
        box[k] = 0;
        d[k] = kMaxLevel + 1;
        D[k] = 0;
        if (i < t.n) {
            key[k] = t.keys[i];
            D[k] = depth[i];
            box[k] = tree_box(t, i);
            d[k] = first_level(t, i, box[k], key[k]);
        }
        const bool starts = d[k] <= D[k];  // never past the last particle
        const int last = min(63, t.n - 1 - (base + ch * 64));
        if (lane == 0) {  // none
            open[ch][0] = kMaxLevel + 1;
            open[ch][1] = 0;
        }
        if (__ballot(starts) == 0) continue;
        int lo = starts ? d[k] : kMaxLevel + 1, hi = starts ? D[k] : 0;
        for (int o = 32; o > 0; o >>= 1) {
            lo = min(lo, __shfl_xor(lo, o, 64));
            hi = max(hi, __shfl_xor(hi, o, 64));
        }
        const int dlast = __builtin_amdgcn_readlane(D[k], last);
        if (lane == 0) {
            open[ch][0] = lo;
            open[ch][1] = dlast;
        }
        for (int l = lo > 1 ? lo : 1; l <= hi; ++l) {
            const uint64_t mc = __ballot(starts && d[k] <= l && l <= D[k]), ml = __ballot(starts && D[k] == l);
            if (lane == 0) {
                cc[ch][l] = __popcll(mc);
                cl[ch][l] = __popcll(ml);
            }
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < kTreeChunks * 32; q += kTreeThreads) {
        const int ch = q >> 5, l = q & 31;
        if (l < max(open[ch][0], 1) || l > open[ch][1]) continue;
        // the first key outside the last particle's cell: by doubling steps, then bisection
        const int last = min(base + ch * 64 + 63, t.n - 1), sh = 3 * (kMaxLevel - l);
        const int bend = box_end(t, tree_box(t, last));
        const uint64_t pre = t.keys[last] >> sh;
        int a = last, step = 1;  // particle a is inside
        int z = bend;            // particle z is outside, or z = bend
        while (a < bend - 1) {
            const int e = a + min(step, bend - 1 - a);
            if ((t.keys[e] >> sh) != pre) {
                z = e;
                break;
            }
            a = e;
            step *= 2;
        }
        while (z - a > 1) {
            const int mid = a + (z - a) / 2;
            if ((t.keys[mid] >> sh) == pre) a = mid;
            else z = mid;
        }
        ends[ch][l] = z;
    }
    if (lane >= 1 && lane <= kMaxLevel && w < 2) {  // exclusive over the runs, from the scan's base
        const int l = lane;
        const size_t row = (size_t)((w ? kMaxLevel : 0) + l - 1) * nblk;
        int run = scan[row + blockIdx.x] + (w ? nleaf0 - scan[(size_t)kMaxLevel * nblk] : t.nbox);
        for (int q = 0; q < kTreeChunks; ++q) {
            int *v = w ? &cl[q][l] : &cc[q][l];
            const int c = *v;
            *v = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int ch = k * (kTreeThreads / 64) + w, c0 = base + ch * 64, i = c0 + lane;
        if (c0 >= t.n) continue;
        const bool valid = i < t.n, starts = valid && d[k] <= D[k];
        // levels this run needs: a beginning cell's parent level to its leaf, every particle's leaf
        int lo = starts ? d[k] - 1 : (valid ? D[k] : kMaxLevel), hi = valid ? D[k] : 0;
        for (int o = 32; o > 0; o >>= 1) {
            lo = min(lo, __shfl_xor(lo, o, 64));
            hi = max(hi, __shfl_xor(hi, o, 64));
        }
        lo = lo > 0 ? lo : 0;
        // cells of level l begun up to this particle, as an index past the last of them
        auto upto = [&](int l) __attribute__((always_inline)) {
            const uint64_t m = __ballot(starts && d[k] <= l && l <= D[k]);
            return l == 0 ? box[k] + 1 : cc[ch][l] + (int)__popcll(m & le);
        };
        int prev = 0, at = upto(lo), leaf = box[k];
        for (int l = lo; l <= hi; ++l) {
            const int next = l < hi ? upto(l + 1) : 0;
            const uint64_t ml = __ballot(starts && D[k] == l), mb = __ballot(valid && d[k] <= l);
            if (valid && D[k] == l) leaf = at - 1;
            if (l == 0) {
                if (starts && d[k] == 0 && D[k] > 0) cells[box[k]].child = next - 1;
            } else if (starts && d[k] <= l && l <= D[k]) {
                const int c = at - 1, sh = 3 * (kMaxLevel - l);
                const int lb = cl[ch][l] + (int)__popcll(ml & lt);  // leaves before this cell
                const uint64_t pre = key[k] >> sh;
                const uint64_t later = mb & ~le;
                const int end = later ? c0 + (int)__ffsll((unsigned long long)later) - 1 : ends[ch][l];
                Cell q;
                q.xln = pack_xln((int)compact3(pre >> 2), l, 0);
                q.iy = (int)compact3(pre >> 1);
                q.iz = (int)compact3(pre);
                q.child = l < D[k] ? next - 1 : -1;
                q.beg = i;
                q.end = end;
                q.parent = prev - 1;
                q.pad = 0;
                cells[c] = q;
                if (l == D[k]) leaves[lb] = c;
                else inner[c - lb] = c;
            }
            prev = at;
            at = next;
        }
        if (valid) leaf_of[i] = leaf;
    }
}

// Child counts of the cells with children: the run of cells from the first child that name
// the cell as their parent.
__global__ void k_child_counts(Cell *__restrict__ cells, int ncell, const int *__restrict__ inner, int ninner)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ninner) return;
    const int c = inner[q], first = cells[c].child;
    int k = 1;
    while (k < 8 && first + k < ncell && cells[first + k].parent == c) ++k;
    cells[c].xln |= k << 26;
}

// Particles in Morton order: wrapped FP64 positions and masses, and FP32 records relative to
// the centre of their leaf (the FP32 form keeps FP64 only for absolute positions and the
// exact cell-centre offsets); the leaf's cube follows from the key and the depth.  Without
// rel: positions and masses only.
__global__ void k_gather(const double *__restrict__ pos, const double *__restrict__ mass,
                         const uint32_t *__restrict__ idx, const uint64_t *__restrict__ keys,
                         const unsigned char *__restrict__ depth, int n, double box, double *__restrict__ xs,
                         double *__restrict__ ys, double *__restrict__ zs, double *__restrict__ ms,
                         int *__restrict__ perm, float4 *__restrict__ rel)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t j = idx[i];
    double x = pos[3 * (size_t)j], y = pos[3 * (size_t)j + 1], z = pos[3 * (size_t)j + 2];
    x = isfinite(x) ? wrap_coord(x, box) : 0.0;
    y = isfinite(y) ? wrap_coord(y, box) : 0.0;
    z = isfinite(z) ? wrap_coord(z, box) : 0.0;
    const double m = mass[j];
    xs[i] = x;
    ys[i] = y;
    zs[i] = z;
    ms[i] = m;
    if (!rel) return;
    perm[i] = (int)j;
    const int l = depth[i];
    const uint64_t pre = keys[i] >> (3 * (kMaxLevel - l));
    const double h = ldexp(box, -l);
    rel[i] = make_float4((float)(x - ((int)compact3(pre >> 2) + 0.5) * h), (float)(y - ((int)compact3(pre >> 1) + 0.5) * h),
                         (float)(z - ((int)compact3(pre) + 0.5) * h), (float)m);
}

static inline int blocks(int64_t n, int b) { return (int)((n + b - 1) / b); }

// Particles of one box ordered by the first 3 `levels` bits of their Morton keys.
int morton_order(MortonSort &s, int n, double box, const double *pos, const double *mass, int levels, int *bad,
                 hipStream_t st)
{
    const size_t nn = (size_t)n;
    int rc = 0;
    for (int b = 0; b < 2 && !rc; ++b) rc = grow(s.keys[b], nn * 8) | grow(s.idx[b], nn * 4);
    if (!rc) rc = grow(s.xs, nn * 8) | grow(s.ys, nn * 8) | grow(s.zs, nn * 8) | grow(s.ms, nn * 8);
    if (rc) return rc;
    s.sorted = 0;
    k_keys<<<blocks(n, 256), 256, 0, st>>>(pos, n, box, ptr<uint64_t>(s.keys[0]), ptr<uint32_t>(s.idx[0]), bad);
    const int first = (63 - 3 * levels) / 8;
    if ((rc = radix_sort(s.keys, s.idx, s.tmp, s.scan_tmp, s.sorted, n, nullptr, 1, first, st))) return rc;
    k_gather<<<blocks(n, 256), 256, 0, st>>>(pos, mass, ptr<uint32_t>(s.idx[s.sorted]), nullptr, nullptr, n, box,
                                             ptr<double>(s.xs), ptr<double>(s.ys), ptr<double>(s.zs), ptr<double>(s.ms),
                                             nullptr, nullptr);
    return hip_check(hipGetLastError(), "particle order");
}

int tree_build(fmm_tree *t, const fmm_params *P, int64_t n64, const double *pos, const double *mass, int nbox,
               const int64_t *hoff, hipStream_t st)
{
    if (n64 < 0 || n64 > (int64_t)1 << 30) return set_error(FMM_ERR_ARG, "n = %lld out of range", (long long)n64);
    if (nbox < 1 || nbox > 65536) return set_error(FMM_ERR_ARG, "nbox = %d out of range", nbox);
    int n = (int)n64;
    t->n = n;
    t->box = P->box;
    t->ncrit = P->n_crit;
    const size_t nn = (size_t)(n > 0 ? n : 1);
    int rc = 0;
    for (int b = 0; b < 2 && !rc; ++b) rc = grow(t->keys[b], nn * 8) | grow(t->idx[b], nn * 4);
    if (!rc) rc = grow(t->xs, nn * 8) | grow(t->ys, nn * 8) | grow(t->zs, nn * 8) | grow(t->ms, nn * 8);
    if (!rc) rc = grow(t->perm, nn * 4) | grow(t->leaf_of, nn * 4) | grow(t->rel32, nn * 16) | grow(t->nearf, nn * 24);
    if (!rc) rc = grow(t->flag, 64 * sizeof(int));
    if (!rc) rc = grow(t->boxoff, (size_t)(nbox + 1) * 4);
    if (rc) return rc;
    t->nbox = nbox;
    t->hboxoff.resize(nbox + 1);
    for (int b = 0; b <= nbox; ++b) t->hboxoff[b] = hoff ? (int)hoff[b] : (b ? n : 0);
    if ((rc = hip_check(hipMemcpyAsync(t->boxoff.p, t->hboxoff.data(), (size_t)(nbox + 1) * 4, hipMemcpyHostToDevice, st),
                        "box offsets")))
        return rc;
    if (!t->host) {
        if (hipHostMalloc((void **)&t->host, kHostInts * sizeof(int), hipHostMallocDefault) != hipSuccess)
            return set_error(FMM_ERR_NOMEM, "pinned host buffer");
    }
    int *bad = ptr<int>(t->flag);
    if ((rc = hip_check(hipMemsetAsync(bad, 0, 4 * sizeof(int), st), "tree flags"))) return rc;
    t->lvl_beg.assign(1, 0);
    if (n == 0) {  // the empty roots
        if ((rc = grow(t->cells, sizeof(Cell) * (size_t)nbox))) return rc;
        k_roots<<<1, 1024, 0, st>>>(ptr<int>(t->boxoff), nbox, P->n_crit, ptr<Cell>(t->cells), nullptr, nullptr, nullptr, nullptr,
                                    nullptr, 0, nullptr);
        t->lvl_beg.push_back(nbox);
        t->nlevel = 1;
        t->ncell = nbox;
        t->nleaf = 0;
        t->leaf_lvl.assign(2, 0);
        return hip_check(hipStreamSynchronize(st), "tree");
    }
    if (!t->bev && hipEventCreateWithFlags(&t->bev, hipEventDisableTiming) != hipSuccess)
        return set_error(FMM_ERR_HIP, "hipEventCreateWithFlags");
    t->sorted = 0;
    k_keys<<<blocks(n, 256), 256, 0, st>>>(pos, n, P->box, ptr<uint64_t>(t->keys[0]), ptr<uint32_t>(t->idx[0]), bad);
    // The sort starts at the key's third digit: bits 16 .. 62 order the particles exactly to
    // level 15 (a level-l octant is decided by key bits 3 (21 - l) .. 3 (21 - l) + 2).  Only
    // a tree that splits a level-15 cell needs the two lowest digits: its arrays are sorted
    // again over every digit (a full LSD sort of the partly sorted arrays).
    constexpr int kPartialDigit = 2, kPartialLevel = 15;
    // small tiles, a run to each wave, where one run after another is what bounds the passes;
    // measured (us a build, tiles of 256 / 1,024 particles): 4,096 particles 112 / 118, 131,072
    // 155 / 166, 524,288 230 / 242, 1,048,576 330 / 330, 2,097,152 446 / 435, 16,777,216 2,880 / 2,743
    const bool small = n <= 1 << 19;
    const int nblk = blocks(n, kTreeThreads * (small ? 1 : 4)), ncount = 2 * kMaxLevel * nblk;
    const int nc = P->n_crit;
    int wexp = 0;  // 2^wexp <= n_crit + 1 < 2^(wexp + 1)
    while (((int64_t)2 << wexp) <= (int64_t)nc + 1) ++wexp;
    int *deep = bad + 2, *nleaf0 = bad + 3, *starts = bad + 8;  // flag area
    int *h = t->host;
    int *scan = nullptr;
    const unsigned char *depth = nullptr;
    TreeIn in{nullptr, ptr<int>(t->boxoff), n, nbox, nc, kPartialLevel};
    for (int first = kPartialDigit;; first = 0) {
        if ((rc = radix_sort(t->keys, t->idx, t->nch, t->scan_tmp, t->sorted, n, ptr<int>(t->boxoff), nbox, first, st)))
            return rc;
        in.keys = ptr<uint64_t>(t->keys[t->sorted]);
        in.lmax = first ? kPartialLevel : kMaxLevel;
        // the sort's other buffers are free: depths in the indices', wide windows in the keys'
        unsigned char *dep = ptr<unsigned char>(t->idx[t->sorted ^ 1]);
        depth = dep;
        const unsigned char *win = nullptr;
        if (nc > kTreeWin && nc < n) {
            const int len = n + nc;
            unsigned char *a = ptr<unsigned char>(t->keys[t->sorted ^ 1]), *b = a + len;
            k_window_levels<<<blocks(len, 256), 256, 0, st>>>(in, a, len);
            for (int k = 0; k < wexp; ++k) {
                k_window_max<<<blocks(len, 256), 256, 0, st>>>(a, b, len, 1 << k);
                unsigned char *c = a;
                a = b;
                b = c;
            }
            win = a;
        }
        if ((rc = grow(t->nch, (size_t)ncount * 2 * sizeof(int)))) return rc;
        int *count = ptr<int>(t->nch);
        scan = count + ncount;
        (small ? k_depth<1> : k_depth<4>)<<<nblk, kTreeThreads, 0, st>>>(in, win, wexp, dep, nblk, count, deep);
        if ((rc = scan_exclusive(count, scan, ncount, nullptr, st, t->scan_tmp))) return rc;
        k_roots<<<1, 1024, 0, st>>>(ptr<int>(t->boxoff), nbox, nc, nullptr, nullptr, nullptr, nleaf0, count, scan, nblk,
                                    starts);
        if ((rc = hip_check(hipMemcpyAsync(h, bad, 64 * sizeof(int), hipMemcpyDeviceToHost, st), "tree sizes")) ||
            (rc = hip_check(hipEventRecord(t->bev, st), "event")))
            return rc;
        // runs while the host reads the sizes and prepares the next launches
        k_gather<<<blocks(n, 256), 256, 0, st>>>(pos, mass, ptr<uint32_t>(t->idx[t->sorted]), in.keys, depth, n, P->box,
                                                 ptr<double>(t->xs), ptr<double>(t->ys), ptr<double>(t->zs),
                                                 ptr<double>(t->ms), ptr<int>(t->perm), ptr<float4>(t->rel32));
        if ((rc = hip_check(hipGetLastError(), "tree")) || (rc = hip_check(hipEventSynchronize(t->bev), "tree"))) return rc;
        if (h[0]) return set_error(FMM_ERR_NAN, "non-finite particle position");
        if (!first || !h[2]) break;
    }
    // level sizes: differences of the scan at the levels' first tiles (modulo 2^32; a level
    // holds at most n cells, all of them may not fit an int)
    const int n0 = h[3], *hs = h + 8;
    int64_t ncell = nbox, nleaf = n0;
    t->lvl_beg.push_back(nbox);
    t->leaf_lvl.assign(1, 0);
    t->leaf_lvl.push_back(n0);
    for (int l = 1; l <= kMaxLevel; ++l) {
        const uint32_t cells = (uint32_t)hs[l] - (uint32_t)hs[l - 1];
        const uint32_t lv = (uint32_t)hs[kMaxLevel + l] - (uint32_t)hs[kMaxLevel + l - 1];
        if (cells == 0) break;
        ncell += cells;
        nleaf += lv;
        if (ncell >= kMaxCells) break;
        t->lvl_beg.push_back((int)ncell);
        t->leaf_lvl.push_back((int)nleaf);
    }
    if (ncell >= kMaxCells) {  // interaction-list entries hold the cell index in 27 bits
        t->n = 0;  // the tree is unusable: later calls see an empty tree, never aliased entries
        t->ncell = t->nleaf = t->nlevel = 0;
        t->lvl_beg.assign(1, 0);
        t->leaf_lvl.assign(1, 0);
        t->stats.n = t->stats.n_cells = t->stats.n_leaves = t->stats.max_level = 0;
        return set_error(FMM_ERR_ARG, "octree exceeds the %d cells an interaction-list entry can address (raise n_crit)",
                         kMaxCells - 1);
    }
    t->nlevel = (int)t->lvl_beg.size() - 1;
    t->ncell = (int)ncell;
    t->nleaf = (int)nleaf;
    const int ninner = t->ncell - t->nleaf;
    if ((rc = grow(t->cells, sizeof(Cell) * (size_t)t->ncell) | grow(t->leaves, (size_t)t->nleaf * 4 + 4) |
              grow(t->inner, (size_t)ninner * 4 + 4)))
        return rc;
    k_roots<<<1, 1024, 0, st>>>(ptr<int>(t->boxoff), nbox, nc, ptr<Cell>(t->cells), ptr<int>(t->leaves),
                                ptr<int>(t->inner), nullptr, nullptr, nullptr, 0, nullptr);
    (small ? k_cells<1> : k_cells<4>)<<<nblk, kTreeThreads, 0, st>>>(in, depth, nblk, scan, n0, ptr<Cell>(t->cells), ptr<int>(t->leaves),
                                           ptr<int>(t->inner), ptr<int>(t->leaf_of));
    if (ninner > 0)
        k_child_counts<<<blocks(ninner, 256), 256, 0, st>>>(ptr<Cell>(t->cells), t->ncell, ptr<int>(t->inner), ninner);
    return hip_check(hipGetLastError(), "tree cells");
}

}  // namespace hfmm
