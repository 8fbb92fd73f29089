// P2P: direct truncated interaction between a sink leaf and the leaves of its P2P list
// (Sec. 2.1 last paragraph; force law of Sec. 2.2):  a_i += m_j f_(1)(r) d, d = x_i - x_j - s box,
// counted iff 0 < r^2 < r_cut^2.
//
// One 64-lane wave per sink leaf.  The sources of up to 64 list entries form one stream
// of slots (a wave prefix sum over the entry sizes), staged 256 slots at a time in LDS.
// A sink of n_A <= C particles (the sink tile, C = 16, 32 or 64, default 32) is held
// floor(64 / n_A) times in the wave; copy g walks slots g, g + G, ... of the staged stream,
// and the copies are summed through LDS at the end.  Larger leaves are processed in
// Morton-ordered chunks of C sink particles, each culled against the box of its own
// particles: chunks of 32 against chunks of 64 culled by the leaf's box, 2M box 8.49 ->
// 7.83 ms at n_crit 48, 16.7M box 56.7 -> 51.6 ms and 134M box 480 -> 430 ms at n_crit 96
// (chunks of 16: 1% slower).
//
// FP64 form: absolute FP64 positions, and for r_cut up to 5 r_s a polynomial for the force law
// too, written about the cutoff so that nothing cancels there (p2p_law.h; beyond that erfc and
// exp of the device math library); sums in FP64.
// FP32 form: FP32 coordinates relative to each particle's leaf centre, the exact
// centre offset c_B + s box - c_A added when staging, and
//   f_(1)(r) = -1/r^3 + S(t)/(8 r_s^3),  t = 2 r^2/r_cut^2 - 1,
// with S(t) = (4/sqrt(pi)) int_0^1 q^2 exp(-v q^2) dq (v = r^2/4r_s^2) replaced by a
// polynomial of degree 9, 10 or 14 fitted on the host, the lowest that meets the FP32
// tolerance at this r_cut / r_s <= 6 (its coefficients carry the factor 1/(8 r_s^3));
// the sum of each staged block is added to a Kahan-compensated per-particle accumulator.
// Both forms: a listed source leaf whose particles' bounding box lies farther than r_cut from
// the sink leaf's box, and any single source particle farther than r_cut from that box, hold
// no pair inside the cutoff and are not staged (the lists themselves are unchanged).
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "expand_impl.h"

namespace hfmm {

struct P2PArgs {
    const Cell *cells;
    const int *leaves;
    int nleaf;
    const int *head;  // P2P list kind: head/cnt offset by ncell already
    const int *cnt;
    const uint32_t *items;
    const int *next;
    const double *xs, *ys, *zs, *ms;
    const float4 *rel;
    double box;
    double *nearf;  // 3 x n SoA
    int n;
    // kP2PSlots lines: [0] listed particle pairs (sum of n_A n_B over P2P leaf pairs), [1]
    // particle pairs evaluated (after the box tests)
    unsigned long long *slots;
    const float4 *bbox;             // per cell: lo, hi of the particles relative to the cell centre
    int first;                      // k_p2p: block b takes sink leaf leaves[first + b]
    const int *err;                 // k_p2p: if non-NULL and non-zero, the lists are void: do nothing
    long long wide_cost;            // leaves of this p2p_cost or more go to k_p2p_wide
    int lcap;                       // last P2P list chunk
    int *wide;                      // [0] their number, [1 ..] their places in `leaves`
};

// Bounding box of each leaf's particles in the FP32 cell-relative frame.
__global__ void k_leaf_bbox(const Cell *__restrict__ cells, const int *__restrict__ leaves, int nleaf,
                            const float4 *__restrict__ rel, float4 *__restrict__ bbox)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nleaf) return;
    int c = leaves[t];
    Cell cc = cells[c];
    float lx = 0, ly = 0, lz = 0, hx = 0, hy = 0, hz = 0;
    if (cc.end > cc.beg) {
        float4 r = rel[cc.beg];
        lx = hx = r.x; ly = hy = r.y; lz = hz = r.z;
        for (int i = cc.beg + 1; i < cc.end; ++i) {
            r = rel[i];
            lx = fminf(lx, r.x); hx = fmaxf(hx, r.x);
            ly = fminf(ly, r.y); hy = fmaxf(hy, r.y);
            lz = fminf(lz, r.z); hz = fmaxf(hz, r.z);
        }
    }
    bbox[2 * (size_t)c] = make_float4(lx, ly, lz, 0.0f);
    bbox[2 * (size_t)c + 1] = make_float4(hx, hy, hz, 0.0f);
}

__device__ __forceinline__ void kahan_add(float &s, float &c, float v)
{
    float y = v - c;
    float t = s + y;
    c = (t - s) - y;
    s = t;
}

constexpr int kStage = 256;  // FP32 form; the FP64 form's 32-byte records are staged 128 at a time
template <bool F64> constexpr int stage_slots() { return F64 ? 128 : kStage; }

// Sink particles per pass over a leaf's list unless fmm_params.p2p_chunk names 16 or 64: a
// leaf of more is processed in Morton-ordered chunks of this many, each tested against the
// box of its own particles.
constexpr int kSinkChunk = 32;

__device__ __forceinline__ float wave_minf(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ float wave_maxf(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Shared memory of one sink leaf's P2P (one 64-lane wave).
template <bool F64> struct P2PShared {
    using V4 = typename std::conditional<F64, double4, float4>::type;
    V4 src[stage_slots<F64>()];
    V4 eoff[64 + 1];        // offset of the entry's records; the last is never read for a slot in use
    int ebase[64], epref[64];  // particle index less slot, first slot of the entry
    int smark[stage_slots<F64>()];
};

template <bool F64> using P2PLaw = typename std::conditional<F64, P2PConst64, P2PConst>::type;

// One sink leaf: its cell and the box of the particles at hand (relative to the cell's centre).
template <bool F64> struct P2PSink {
    Cell ca;
    double box, hA, cax, cay, caz;  // FP64 form: times scale, as the rest
    // FP64 form: along an axis where the leaf lies in the box's last quarter, its coordinates
    // count from the box's far face.  An image x + box would be rounded to the last place of
    // box, while x - box of a particle at box / 2 or above is exact; the particles below box / 2,
    // for which it is not, are a quarter of the box away.  Wider leaves keep their coordinates:
    // they hold particles nearer to such ones, or such ones themselves.
    double Ox = 0.0, Oy = 0.0, Oz = 0.0;
    // FP64 form: the boxes are FP32 and relative to their leaves, so their rounding grows with
    // the leaves' sides, however small the cutoff: the tests' margin does too
    float cutA = 0.0f;
    float4 alo, ahi;

    __device__ __forceinline__ P2PSink(const P2PArgs &a, const P2PLaw<F64> &k, int A)
    {
        ca = a.cells[A];
        box = a.box;
        if constexpr (F64) box *= k.scale;
        hA = ldexp(box, -cell_level(ca));
        cax = (cell_ix(ca) + 0.5) * hA;
        cay = (ca.iy + 0.5) * hA;
        caz = (ca.iz + 0.5) * hA;
        alo = a.bbox[2 * (size_t)A];
        ahi = a.bbox[2 * (size_t)A + 1];
        if constexpr (F64) {
            scale_box(k);
            cutA = k.cut + 1e-6f * (float)hA;
            const int q = cell_level(ca) - 2;
            Ox = q >= 0 && cell_ix(ca) >> q == 3 ? box : 0.0;
            Oy = q >= 0 && ca.iy >> q == 3 ? box : 0.0;
            Oz = q >= 0 && ca.iz >> q == 3 ? box : 0.0;
        }
    }

    __device__ __forceinline__ void scale_box(const P2PConst64 &k)
    {
        alo = make_float4(alo.x * k.scale32, alo.y * k.scale32, alo.z * k.scale32, 0.0f);
        ahi = make_float4(ahi.x * k.scale32, ahi.y * k.scale32, ahi.z * k.scale32, 0.0f);
    }

    // the box of the ns particles from `first` (one chunk of the leaf)
    __device__ __forceinline__ void chunk_box(const P2PArgs &a, const P2PLaw<F64> &k, int first, int ns, int lane)
    {
        const float4 me = a.rel[first + (lane < ns ? lane : 0)];
        alo = make_float4(wave_minf(me.x), wave_minf(me.y), wave_minf(me.z), 0.0f);
        ahi = make_float4(wave_maxf(me.x), wave_maxf(me.y), wave_maxf(me.z), 0.0f);
        if constexpr (F64) scale_box(k);
    }

    // sink particle i in the pair loop's coordinates
    template <class R>
    __device__ __forceinline__ void load(const P2PArgs &a, const P2PLaw<F64> &k, int i, R &xi, R &yi, R &zi) const
    {
        if constexpr (F64) {
            xi = fma(a.xs[i], k.scale, -Ox);
            yi = fma(a.ys[i], k.scale, -Oy);
            zi = fma(a.zs[i], k.scale, -Oz);
        } else {
            float4 me = a.rel[i];
            xi = me.x; yi = me.y; zi = me.z;
        }
        // the sink's load ends here: left to its first use, inside the pair loop, it would make
        // that loop wait for the next stage's records too
        asm volatile("" : "+v"(xi), "+v"(yi), "+v"(zi));
    }

    // List entry `it` of this lane: its record offset into eoff[lane], its first particle and
    // particle count; cntj is 0 if its box lies beyond the cutoff of the sink's.
    template <class V4>
    __device__ __forceinline__ void entry(const P2PArgs &a, const P2PLaw<F64> &k, uint32_t it, V4 *eoff, int lane,
                                          int &cntj, int &listed, int &jbeg) const
    {
        int s = (int)(it & 31);
        Cell cb = a.cells[it >> 5];
        cntj = listed = cb.end - cb.beg;
        jbeg = cb.beg;
        double shx = (double)(s / 9 - 1) * box, shy = (double)((s / 3) % 3 - 1) * box, shz = (double)(s % 3 - 1) * box;
        // exact in FP64: dyadic centres and integer image shifts
        double hB = ldexp(box, -cell_level(cb));
        const float ox = (float)((cell_ix(cb) + 0.5) * hB + shx - cax);
        const float oy = (float)((cb.iy + 0.5) * hB + shy - cay);
        const float oz = (float)((cb.iz + 0.5) * hB + shz - caz);
        if constexpr (F64) eoff[lane] = make_double4(shx - Ox, shy - Oy, shz - Oz, 0.0);
        else eoff[lane] = make_float4(ox, oy, oz, 0.0f);
        // gap between the two boxes; the margin covers FP32 rounding many times over
        float4 blo = a.bbox[2 * (size_t)(it >> 5)], bhi = a.bbox[2 * (size_t)(it >> 5) + 1];
        if constexpr (F64) {
            const float c = k.scale32;
            blo.x *= c; blo.y *= c; blo.z *= c;
            bhi.x *= c; bhi.y *= c; bhi.z *= c;
        }
        const float gx = fmaxf(0.0f, fmaxf(alo.x - (bhi.x + ox), (blo.x + ox) - ahi.x));
        const float gy = fmaxf(0.0f, fmaxf(alo.y - (bhi.y + oy), (blo.y + oy) - ahi.y));
        const float gz = fmaxf(0.0f, fmaxf(alo.z - (bhi.z + oz), (blo.z + oz) - ahi.z));
        float far2;
        if constexpr (F64) {
            const float cut = cutA + 1e-6f * (float)hB;
            far2 = cut * cut;
        } else {
            far2 = k.rc2 * 1.0001f;
        }
        if (gx * gx + gy * gy + gz * gz > far2) cntj = 0;
    }
};

// Source records of one stage, a lane's kPer slots, in registers: loaded one stage ahead, so
// their latency is covered by the pair work of the current stage.
template <bool F64> struct P2PFetch {
    using V4 = typename std::conditional<F64, double4, float4>::type;
    static constexpr int kPer = stage_slots<F64>() / 64;
    V4 rv[kPer];
    int ev[kPer];  // list entry of each slot; 64: past the end

    // Slots [sbase, sbase + stage) of the list block in m (its ne entries, `total` slots).
    // Slot -> list entry: each entry marks the slot it starts at (the largest entry wins, so
    // entries left empty by the box test are skipped), and a max-scan over the slots carries
    // the marks forward.  Lane l owns slots kPer l .. kPer l + kPer - 1.  efirst: the entry
    // that holds slot sbase unless one starts there (the marks then supply it).
    __device__ __forceinline__ void fetch(const P2PArgs &a, const P2PShared<F64> &m, int *smark, int ne, int total,
                                          int sbase, int efirst, int lane)
    {
        constexpr int kStage = stage_slots<F64>();
        const int nraw = min(kStage, total - sbase);
#pragma unroll
        for (int u = 0; u < kPer; ++u) smark[kPer * lane + u] = 0;
        wave_sync();
        if (lane < ne) {
            const int st = m.epref[lane] - sbase;
            if (st >= 0 && st < kStage) atomicMax(&smark[st], lane + 1);
        }
        wave_sync();
        int mrun[kPer], mx = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            mx = max(mx, smark[kPer * lane + u]);
            mrun[u] = mx;
        }
        const int incl = wave_incl_max(mx);
        const int prev = wave_shift_up1(incl);
        const int base = max(prev, efirst + 1);
        // every address first, then the loads back to back: a load under its own
        // branch waits for the one before it (lanes past the end load record 0)
        int jv[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) jv[u] = m.ebase[max(base, mrun[u]) - 1];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int q = kPer * lane + u;
            ev[u] = q < nraw ? max(base, mrun[u]) - 1 : 64;
            jv[u] = q < nraw ? jv[u] + sbase + q : 0;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if constexpr (F64) rv[u] = make_double4(a.xs[jv[u]], a.ys[jv[u]], a.zs[jv[u]], a.ms[jv[u]]);
            else rv[u] = a.rel[jv[u]];
        }
    }

    // The fetched sources, moved by their entries' offsets, into src; returns their number.
    // A source particle farther than r_cut from the sink's box meets no sink particle inside
    // the cutoff: it is not staged (ballot compaction).
    __device__ __forceinline__ int stage(const P2PSink<F64> &sk, const P2PLaw<F64> &k, const V4 *eoff, V4 *src,
                                         uint64_t lt) const
    {
        int nst = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const V4 eo = eoff[ev[u]];
            V4 sv;
            sv.w = rv[u].w;
            float px, py, pz, far2;  // the source relative to the sink leaf's centre
            if constexpr (F64) {
                sv.x = fma(rv[u].x, k.scale, eo.x);
                sv.y = fma(rv[u].y, k.scale, eo.y);
                sv.z = fma(rv[u].z, k.scale, eo.z);
                px = (float)(sv.x - (sk.cax - sk.Ox));
                py = (float)(sv.y - (sk.cay - sk.Oy));
                pz = (float)(sv.z - (sk.caz - sk.Oz));
                far2 = sk.cutA * sk.cutA;
            } else {
                sv.x = rv[u].x + eo.x;
                sv.y = rv[u].y + eo.y;
                sv.z = rv[u].z + eo.z;
                px = sv.x; py = sv.y; pz = sv.z;
                far2 = k.rc2 * 1.0001f;
            }
            const float gx = fmaxf(0.0f, fmaxf(sk.alo.x - px, px - sk.ahi.x));
            const float gy = fmaxf(0.0f, fmaxf(sk.alo.y - py, py - sk.ahi.y));
            const float gz = fmaxf(0.0f, fmaxf(sk.alo.z - pz, pz - sk.ahi.z));
            const bool keep = ev[u] < 64 && gx * gx + gy * gy + gz * gz <= far2;
            const uint64_t km = __ballot(keep);
            if (keep) src[nst + __popcll(km & lt)] = sv;
            nst += __popcll(km);
        }
        return nst;
    }
};

// FP32 form: the force of the staged sources g, g + G, ... on one sink particle.
// POLY (polynomial split): f_(1) = -1/r^3 + 5/(2 r_c^3) - 3 r^2/(2 r_c^5) evaluated as
// -(1-x)^2 (1 + 2x + 3x^2 + 3x^3/2) / r^3, x = r / r_c: the three terms cancel near r_cut in
// FP32, the factored form does not.
template <bool POLY, int NPC>
__device__ __forceinline__ void p2p_sum32(const P2PConst &k, const float4 *src, int nst, int g, int G, float xi, float yi,
                                          float zi, float &px, float &py, float &pz)
{
    px = py = pz = 0.0f;
    // the leading coefficient as a vector operand: each Horner step then reads a single scalar
    float clead = k.c[NPC - 1];
    asm volatile("" : "+v"(clead));
    auto pair = [&](const float4 s) __attribute__((always_inline)) {
        const float dx = xi - s.x, dy = yi - s.y, dz = zi - s.z;
        // a particle meets itself (and exact duplicates) at d = 0: the 1e-20 added to r^2 keeps
        // w finite, so w d = 0 without a separate r > 0 test; for any other pair it is far
        // below r^2's rounding
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, 1e-20f)));
        const float rinv = __frsqrt_rn(r2);
        float f1;
        if constexpr (POLY) {
            const float x = r2 * rinv * k.c[0], omx = 1.0f - x;
            const float q = fmaf(fmaf(fmaf(1.5f, x, 3.0f), x, 2.0f), x, 1.0f);
            f1 = -(omx * omx) * q * (rinv * rinv * rinv);
        } else {
            const float t = fmaf(r2, k.two_over_rc2, -1.0f);
            float S = clead;  // S(t) / (8 r_s^3)
#pragma unroll
            for (int c = NPC - 2; c >= 0; --c) S = fmaf(S, t, k.c[c]);
            f1 = fmaf(-rinv * rinv, rinv, S);
        }
        const float w = r2 < k.rc2 ? s.w * f1 : 0.0f;
        px = fmaf(w, dx, px);
        py = fmaf(w, dy, py);
        pz = fmaf(w, dz, pz);
    };
    // four sources per step, read two at a time
    const float4 *sp = src + g;
    const float4 *const send = src + nst;
    for (; sp + 3 * G < send; sp += 4 * G) {
        const float4 s0 = sp[0], s1 = sp[G];
        pair(s0);
        pair(s1);
        const float4 s2 = sp[2 * G], s3 = sp[3 * G];
        pair(s2);
        pair(s3);
    }
    for (; sp < send; sp += G) pair(sp[0]);
}

// FP64 form: the same, added to ax, ay, az.
template <int NPC>
__device__ __forceinline__ void p2p_sum64(const P2PConst64 &k, const double4 *src, int nst, int g, int G, double xi,
                                          double yi, double zi, double &ax, double &ay, double &az)
{
    auto pair = [&](const double4 s) __attribute__((always_inline)) {
        const double dx = xi - s.x, dy = yi - s.y, dz = zi - s.z;
        const double r2 = dx * dx + dy * dy + dz * dz;
        const double w = law64_weight<NPC>(k, r2, s.w, __builtin_amdgcn_rsq(r2));
        ax += w * dx;
        ay += w * dy;
        az += w * dz;
    };
    int q = g;
    for (; q + G < nst; q += 2 * G) {  // two sources per step
        const double4 s0 = src[q], s1 = src[q + G];
        pair(s0);
        pair(s1);
    }
    if (q < nst) pair(src[q]);
}

// The copies of each sink particle (red[copy ns + particle]) summed and written.
template <bool F64>
__device__ __forceinline__ void p2p_write(const P2PArgs &a, const P2PLaw<F64> &k, const double (*red)[3], int first,
                                          int ns, int G, int lane)
{
    if (lane >= ns) return;
    double tx = 0, ty = 0, tz = 0;
    for (int q = 0; q < G; ++q) {
        tx += red[q * ns + lane][0];
        ty += red[q * ns + lane][1];
        tz += red[q * ns + lane][2];
    }
    if constexpr (F64) {  // masses over lengths squared
        tx = tx * k.scale * k.scale;
        ty = ty * k.scale * k.scale;
        tz = tz * k.scale * k.scale;
    }
    const int o = first + lane;
    a.nearf[o] = tx;
    a.nearf[(size_t)a.n + o] = ty;
    a.nearf[2 * (size_t)a.n + o] = tz;
}

__device__ __forceinline__ void p2p_count(const P2PArgs &a, int li, unsigned long long npairs, unsigned long long nevald)
{
    unsigned long long *c = a.slots + (size_t)(li % kP2PSlots) * kSlotWords;
    atomicAdd(&c[0], npairs);
    atomicAdd(&c[1], nevald);
}

// What a sink leaf costs one wave: list entries times passes over the list.
template <int CHUNK> __device__ __forceinline__ long long p2p_cost(int nA, int nlist)
{
    return (long long)nlist * ((nA + CHUNK - 1) / CHUNK);
}

// P2P of sink leaf `leaves[li]` by one wave (leaves of a.wide_cost or more are left to
// p2p_leaf_wide).
// CHUNK: the sink tile (16, 32 or 64 particles), a compile-time constant: a tile read at
// run time (from P2PConst, or as an extra kernel argument) changed the register allocation
// of the pair loop and cost 0.8-1.1% of the 134M box's P2P time.
template <bool F64, bool POLY, int NPC, int CHUNK>
__device__ __forceinline__ void p2p_leaf(const P2PArgs &a, const P2PLaw<F64> &k, int li, P2PShared<F64> &sh)
{
    constexpr int kStage = stage_slots<F64>();
    using R = typename std::conditional<F64, double, float>::type;
    const int lane = threadIdx.x;
    const uint64_t lt = (1ull << lane) - 1ull;
    const int A = a.leaves[li];
    P2PSink<F64> sk(a, k, A);
    const int nA = sk.ca.end - sk.ca.beg;
    const int nlist = a.cnt[A];
    if (p2p_cost<CHUNK>(nA, nlist) >= a.wide_cost) return;
    unsigned long long npairs = 0, nevald = 0;

    for (int ib = 0; ib < nA; ib += CHUNK) {
        const int ns = min(CHUNK, nA - ib);
        const int G = 64 / ns, g = lane / ns, si = lane - g * ns;
        if (nA > CHUNK) sk.chunk_box(a, k, sk.ca.beg + ib, ns, lane);
        const bool valid = g < G;
        R xi, yi, zi;
        sk.load(a, k, sk.ca.beg + ib + (valid ? si : 0), xi, yi, zi);
        double ax = 0, ay = 0, az = 0;              // FP64 form
        float sx = 0, sy = 0, sz = 0, cx = 0, cy = 0, cz = 0;  // FP32 form (Kahan)
        // the list is read a chunk ahead: the next chunk's items are on their way while the
        // current chunk's sources are summed
        int chunk = a.head[A];
        uint32_t it = lane < nlist ? a.items[(size_t)chunk * kChunk + lane] : 0u;
        for (int eb = 0; eb < nlist; eb += 64) {
            const int ne = min(64, nlist - eb);
            const bool more = eb + 64 < nlist;
            int nchunk = 0;
            if (more) nchunk = a.next[chunk];
            int cntj = 0, listed = 0, jbeg = 0;
            if (lane < ne) sk.entry(a, k, it, sh.eoff, lane, cntj, listed, jbeg);
            const int incl = wave_incl_sum(cntj);
            if (lane < ne) {
                sh.epref[lane] = incl - cntj;
                sh.ebase[lane] = jbeg - (incl - cntj);
            }
            if (more) {
                chunk = nchunk;
                it = lane < nlist - eb - 64 ? a.items[(size_t)chunk * kChunk + lane] : 0u;
            }
            const int total = __builtin_amdgcn_readlane(incl, 63);
            const int ltot = __builtin_amdgcn_readlane(wave_incl_sum(listed), 63);
            npairs += (unsigned long long)ns * (unsigned)ltot;
            wave_sync();
            P2PFetch<F64> f;
            if (total > 0) f.fetch(a, sh, sh.smark, ne, total, 0, 0, lane);
            for (int sb = 0; sb < total; sb += kStage) {
                const int nst = f.stage(sk, k, sh.eoff, sh.src, lt);
                if (sb + kStage < total)
                    f.fetch(a, sh, sh.smark, ne, total, sb + kStage, __builtin_amdgcn_readlane(f.ev[f.kPer - 1], 63), lane);
                nevald += (unsigned long long)ns * (unsigned)nst;
                wave_sync();
                if (valid) {
                    if constexpr (F64) {
                        p2p_sum64<NPC>(k, sh.src, nst, g, G, xi, yi, zi, ax, ay, az);
                    } else {
                        float px, py, pz;
                        p2p_sum32<POLY, NPC>(k, sh.src, nst, g, G, xi, yi, zi, px, py, pz);
                        kahan_add(sx, cx, px);
                        kahan_add(sy, cy, py);
                        kahan_add(sz, cz, pz);
                    }
                }
                wave_sync();
            }
        }
        if constexpr (!F64) {
            ax = (double)sx - (double)cx;
            ay = (double)sy - (double)cy;
            az = (double)sz - (double)cz;
        }
        double(*red)[3] = reinterpret_cast<double(*)[3]>(&sh.src[0]);  // staging area is free here
        red[lane][0] = ax;
        red[lane][1] = ay;
        red[lane][2] = az;
        wave_sync();
        p2p_write<F64>(a, k, red, sk.ca.beg + ib, ns, G, lane);
        wave_sync();
    }
    if (lane == 0) p2p_count(a, li, npairs, nevald);
}

// P2P of one sink leaf by a workgroup of kWide waves, for leaves so costly that one wave
// would outlast all others.  Each wave reads the entries of one list block of 64; the blocks'
// stages, as the one-wave form cuts them, are then dealt to the waves in turn.  FP32 form: the
// stages' sums go through LDS and wave 0 adds them in the one-wave form's order, so the
// results are the same bit for bit; FP64 form: each wave sums its stages, the waves' sums are
// added in order.
constexpr int kWide = 8;
constexpr int kWideIds = 512;  // list blocks whose chunks are looked up at a time
template <bool F64> struct P2PWideShared {
    P2PShared<F64> w[kWide];
    int tot[kWide], ids[kWideIds];
    float sums[2][F64 ? 1 : kWide][3][64];
};

template <bool F64, bool POLY, int NPC, int CHUNK>
__device__ __forceinline__ void p2p_leaf_wide(const P2PArgs &a, const P2PLaw<F64> &k, int li, P2PWideShared<F64> &ws)
{
    constexpr int kStage = stage_slots<F64>();
    using R = typename std::conditional<F64, double, float>::type;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    const int A = a.leaves[li];
    P2PSink<F64> sk(a, k, A);
    P2PShared<F64> &sh = ws.w[w];
    const int nA = sk.ca.end - sk.ca.beg;
    const int nlist = a.cnt[A], nblk = (nlist + 63) / 64;
    unsigned long long npairs = 0, nevald = 0;
    for (int ib = 0; ib < nA; ib += CHUNK) {
        const int ns = min(CHUNK, nA - ib);
        const int G = 64 / ns, g = lane / ns, si = lane - g * ns;
        if (nA > CHUNK) sk.chunk_box(a, k, sk.ca.beg + ib, ns, lane);
        const bool valid = g < G;
        R xi, yi, zi;
        sk.load(a, k, sk.ca.beg + ib + (valid ? si : 0), xi, yi, zi);
        double ax = 0, ay = 0, az = 0;
        float sx = 0, sy = 0, sz = 0, cx = 0, cy = 0, cz = 0;  // FP32 form: wave 0
        int cur = a.head[A];
        for (int b0 = 0; b0 < nblk; b0 += kWide) {
            if (b0 % kWideIds == 0) {
                // the chunks of the next list blocks: a wave writes its chunks in runs, so 64
                // links read at once usually settle as many blocks
                __syncthreads();
                if (w == 0) {
                    const int need = min(kWideIds, nblk - b0);
                    for (int pos = 0; pos < need;) {
                        const int v = cur + lane <= a.lcap ? a.next[cur + lane] : -1;
                        const uint64_t brk = __ballot(v != cur + lane + 1);
                        const int run = brk ? (int)__ffsll((unsigned long long)brk) : 64;  // chunks cur .. cur + run - 1
                        const int n = min(run, need - pos);
                        if (lane < n) ws.ids[pos + lane] = cur + lane;
                        pos += n;
                        cur = __builtin_amdgcn_readlane(v, n - 1);
                    }
                }
                __syncthreads();
            }
            // entries of this wave's list block
            const int b = b0 + w;
            int total = 0;
            if (b < nblk) {
                const int ne = min(64, nlist - 64 * b);
                int cntj = 0, listed = 0, jbeg = 0;
                if (lane < ne)
                    sk.entry(a, k, a.items[(size_t)ws.ids[b % kWideIds] * kChunk + lane], sh.eoff, lane, cntj, listed, jbeg);
                const int incl = wave_incl_sum(cntj);
                if (lane < ne) {
                    sh.epref[lane] = incl - cntj;
                    sh.ebase[lane] = jbeg - (incl - cntj);
                }
                total = __builtin_amdgcn_readlane(incl, 63);
                npairs += (unsigned long long)ns * (unsigned)__builtin_amdgcn_readlane(wave_incl_sum(listed), 63);
            }
            if (lane == 0) ws.tot[w] = total;
            __syncthreads();
            int nstage = 0;
#pragma unroll
            for (int v = 0; v < kWide; ++v) nstage += (ws.tot[v] + kStage - 1) / kStage;
            nstage = __builtin_amdgcn_readfirstlane(nstage);
            // stage j of these blocks: its block and first slot, fetched into f
            P2PFetch<F64> f;
            int fb = 0;
            auto fetch = [&](int j) __attribute__((always_inline)) {
                int first = 0, v = 0;
                for (; v < kWide - 1; ++v) {
                    const int n = (ws.tot[v] + kStage - 1) / kStage;
                    if (j < first + n) break;
                    first += n;
                }
                fb = __builtin_amdgcn_readfirstlane(v);
                const int sbase = (j - first) * kStage, ne = min(64, nlist - 64 * (b0 + fb)), tot = ws.tot[fb];
                // the entry that holds the first slot: the last one that begins at or before it
                const uint64_t at = __ballot(lane < ne && ws.w[fb].epref[lane] <= sbase);
                f.fetch(a, ws.w[fb], sh.smark, ne, tot, sbase, 63 - (int)__clzll((long long)at), lane);
            };
            if (w < nstage) fetch(w);
            const int rounds = (nstage + kWide - 1) / kWide;
            for (int q = 0; q < rounds; ++q) {
                const int j = q * kWide + w;
                float px = 0, py = 0, pz = 0;
                if (j < nstage) {
                    const int nst = f.stage(sk, k, ws.w[fb].eoff, sh.src, lt);
                    if (j + kWide < nstage) fetch(j + kWide);
                    nevald += (unsigned long long)ns * (unsigned)nst;
                    wave_sync();
                    if (valid) {
                        if constexpr (F64) p2p_sum64<NPC>(k, sh.src, nst, g, G, xi, yi, zi, ax, ay, az);
                        else p2p_sum32<POLY, NPC>(k, sh.src, nst, g, G, xi, yi, zi, px, py, pz);
                    }
                    wave_sync();
                }
                if constexpr (!F64) {
                    ws.sums[q & 1][w][0][lane] = px;
                    ws.sums[q & 1][w][1][lane] = py;
                    ws.sums[q & 1][w][2][lane] = pz;
                    __syncthreads();  // the other half of the sums is rewritten only after the next one
                    if (w == 0 && valid)
                        for (int v = 0; v < min(kWide, nstage - q * kWide); ++v) {
                            kahan_add(sx, cx, ws.sums[q & 1][v][0][lane]);
                            kahan_add(sy, cy, ws.sums[q & 1][v][1][lane]);
                            kahan_add(sz, cz, ws.sums[q & 1][v][2][lane]);
                        }
                }
            }
            __syncthreads();  // the entries are read to the end
        }
        if constexpr (!F64) {
            ax = (double)sx - (double)cx;
            ay = (double)sy - (double)cy;
            az = (double)sz - (double)cz;
        }
        double(*red)[3] = reinterpret_cast<double(*)[3]>(&sh.src[0]);
        red[lane][0] = ax;
        red[lane][1] = ay;
        red[lane][2] = az;
        __syncthreads();
        if (w == 0) {
            if constexpr (F64) {
                for (int v = 1; v < kWide; ++v) {
                    const double(*o)[3] = reinterpret_cast<const double(*)[3]>(&ws.w[v].src[0]);
                    for (int c = 0; c < 3; ++c) red[lane][c] += o[lane][c];
                }
                wave_sync();
            }
            p2p_write<F64>(a, k, red, sk.ca.beg + ib, ns, G, lane);
        }
        __syncthreads();
    }
    if (lane == 0) p2p_count(a, li, npairs, nevald);
}

// FP32 form: bound by FP32 issue, 25 operations a pair; the records of a stage and the items
// of the next list chunk are loaded ahead, every load of a stage issued before the first wait
// (a load under its own branch waited for the one before it, and the sink's own load for all
// of them: 300,007 particles, polynomial split, step 3.50 -> 3.33 ms; 2M 8.13 -> 8.01 ms; 64-box
// forest 11.77 -> 11.46 ms).
// FP64 form: bound by FP64 issue, 49 vector operations a pair with 19 coefficients (41 of them
// FP64; the cancelling form of the law takes 48: 262,144 clustered step 1.73 ms with either, a
// uniform box that is P2P nearly alone 1.18 against 1.23) against well over 200 of erfc, exp, the square root and the division, on the pairs the box
// tests leave (62% of the listed ones on the 2M box) at four waves per SIMD instead of three:
// uniform 32^3 step 1.21 -> 0.83 ms, 262,144 clustered step 9.0 -> 4.5 ms with one wave per leaf.
template <bool F64, bool POLY, int NPC, int CHUNK>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(F64 ? (NPC ? 4 : 2) : 5))) void k_p2p(P2PArgs a,
                                                                                                   P2PLaw<F64> k)
{
    __shared__ P2PShared<F64> sh;
    if (a.err && *a.err) return;  // the traversal overflowed: it reruns, and so does P2P
    p2p_leaf<F64, POLY, NPC, CHUNK>(a, k, a.first + xcd_order(blockIdx.x, gridDim.x), sh);
}

// The leaves of a.wide_cost or more, in any order.
template <int CHUNK> __global__ __launch_bounds__(64) void k_p2p_wide_select(P2PArgs a)
{
    const int li = blockIdx.x * 64 + threadIdx.x;
    if (li >= a.nleaf) return;
    const int A = a.leaves[li];
    if (p2p_cost<CHUNK>(a.cells[A].end - a.cells[A].beg, a.cnt[A]) >= a.wide_cost) a.wide[1 + atomicAdd(a.wide, 1)] = li;
}

template <bool F64, bool POLY, int NPC, int CHUNK>
__global__ __launch_bounds__(64 * kWide) __attribute__((amdgpu_waves_per_eu(F64 ? 2 : 4))) void k_p2p_wide(P2PArgs a,
                                                                                                     P2PLaw<F64> k)
{
    __shared__ P2PWideShared<F64> sh;
    const int n = a.wide[0];
    for (int h = blockIdx.x; h < n; h += gridDim.x) {
        p2p_leaf_wide<F64, POLY, NPC, CHUNK>(a, k, a.wide[1 + h], sh);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Persistent fused P2P + M2L (FP32, plain MAC): the grid holds as many 64-lane blocks as
// fit on the device at once; each block pulls items from one device counter until the
// queue is empty: first the sink leaves (P2P), then the 64-pair blocks of the flattened
// M2L array.  One launch covers both stages of every box of a forest, so no stage waits
// for the tail of another and no launch boundary falls between them.
template <bool POLY, int NPC, int P>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(P >= 7 ? 2 : (P >= 5 ? 3 : 4)))) void k_p2p_m2l_persist(
    P2PArgs a, P2PConst k, const int2 *__restrict__ pairs, int64_t npair, const float *__restrict__ M,
    float *__restrict__ L, Split sp, int stride, int *__restrict__ queue)
{
    __shared__ union {
        P2PShared<false> p;
        M2LPairShared<P, float> m;
    } sh;
    const int nleaf = a.nleaf;
    const int total = nleaf + (int)((npair + 63) / 64);
    for (;;) {
        int item = 0;
        if (threadIdx.x == 0) item = atomicAdd(queue, 1);
        item = __builtin_amdgcn_readfirstlane(__shfl(item, 0, 64));
        if (item >= total) break;
        if (item < nleaf) p2p_leaf<false, POLY, NPC, kSinkChunk>(a, k, item, sh.p);
        else m2l_pairs_block<P, float>(a.cells, pairs, npair, M, L, a.box, sp, stride, item - nleaf, sh.m);
        __syncthreads();  // the block's shared memory is reused by the next item
    }
}

// ---------------------------------------------------------------------------
// host: fit of S(t) on [-1, 1] at Chebyshev points (interpolation, solved in FP64)

static double S_of_v(double v)
{
    // S(v) = (erf(u) - 2u/sqrt(pi) e^{-u^2}) / u^3, u = sqrt(v); series near 0
    if (v < 0.09) {
        double s = 0, term = 1;  // sum (-1)^k v^k / (k! (2k+3))
        for (int k = 0; k < 30; ++k) {
            s += term / (2 * k + 3);
            term *= -v / (k + 1);
        }
        return 4.0 / sqrt(M_PI) * s;
    }
    double u = sqrt(v);
    return (erf(u) - 2.0 * u / sqrt(M_PI) * exp(-v)) / (u * u * u);
}

// Interpolation of S at the m Chebyshev points of t in [-1, 1] (solved in FP64), the
// coefficients of t^0 .. t^(m-1) returned in FP64.
static void fit_S(double vcut, int m, double *coef)
{
    double Amat[kP2PPolyMax][kP2PPolyMax + 1];
    for (int i = 0; i < m; ++i) {
        double t = cos(M_PI * (i + 0.5) / m);
        double v = (t + 1.0) * 0.5 * vcut;
        double pw = 1.0;
        for (int j = 0; j < m; ++j) { Amat[i][j] = pw; pw *= t; }
        Amat[i][m] = S_of_v(v);
    }
    for (int c = 0; c < m; ++c) {  // Gaussian elimination with partial pivoting
        int piv = c;
        for (int r = c + 1; r < m; ++r)
            if (fabs(Amat[r][c]) > fabs(Amat[piv][c])) piv = r;
        for (int j = 0; j <= m; ++j) { double tmp = Amat[c][j]; Amat[c][j] = Amat[piv][j]; Amat[piv][j] = tmp; }
        for (int r = 0; r < m; ++r) {
            if (r == c) continue;
            double f = Amat[r][c] / Amat[c][c];
            for (int j = c; j <= m; ++j) Amat[r][j] -= f * Amat[c][j];
        }
    }
    for (int j = 0; j < m; ++j) coef[j] = Amat[j][m] / Amat[j][j];
}

// Largest error of the fit, with its coefficients rounded to FP32, in r^3 f_(1) = S u^3 - 1
// (u = r / 2 r_s): the pair force's error relative to the Newtonian one, on 4001 points.
static double fit_error(double vcut, int m, const double *coef)
{
    double worst = 0.0;
    for (int i = 0; i <= 4000; ++i) {
        const double t = -1.0 + i / 2000.0, v = (t + 1.0) * 0.5 * vcut;
        double S = (double)(float)coef[m - 1];
        for (int j = m - 2; j >= 0; --j) S = S * t + (double)(float)coef[j];
        const double e = fabs(S - S_of_v(v)) * v * sqrt(v);
        worst = e > worst ? e : worst;
    }
    return worst;
}

// Force-law constants.  FP32 form, Gaussian split: the lowest polynomial length of 10, 11, 15 whose
// checked error is at most kP2PFitTol; returns FMM_ERR_ARG for r_cut > kP2PMaxCut r_s (FP32
// cancellation near the cutoff) or if no fit meets the tolerance.  The last fit is cached
// (same vcut, same result).
int p2p_setup(const fmm_params *P, P2PConst &k)
{
    static std::mutex mu;
    static double cached_vcut = -1.0;
    static int cached_m = 0;
    static double cached[kP2PPolyMax];
    const double vcut = (P->r_cut * P->r_cut) / (4.0 * P->r_s * P->r_s);
    double coef[kP2PPolyMax] = {0};
    int m = 0;
    if (P->precision == 1 && P->split == 0) {  // the FP64 form has its own law (p2p_law.h) and no limit
        if (P->r_cut > kP2PMaxCut * P->r_s)
            return set_error(FMM_ERR_ARG, "precision 1 supports r_cut <= %.0f r_s (r_cut / r_s = %.3g): beyond it the "
                                          "FP32 pair force loses accuracy near the cutoff; use precision 0",
                             kP2PMaxCut, P->r_cut / P->r_s);
        std::lock_guard<std::mutex> lk(mu);
        if (vcut != cached_vcut) {
            cached_m = 0;
            for (int mm : {10, 11, 15}) {
                fit_S(vcut, mm, cached);
                if (fit_error(vcut, mm, cached) <= kP2PFitTol) {
                    cached_m = mm;
                    break;
                }
            }
            cached_vcut = vcut;
        }
        m = cached_m;
        for (int j = 0; j < m; ++j) coef[j] = cached[j];
        if (m == 0)
            return set_error(FMM_ERR_ARG, "precision 1: no polynomial of degree <= 14 meets the FP32 force-law "
                                          "tolerance at r_cut / r_s = %.3g; use precision 0", P->r_cut / P->r_s);
    }
    // the kernel evaluates S(t) / (8 r_s^3): the factor is folded into the coefficients
    const double inv8rs3 = 1.0 / (8.0 * P->r_s * P->r_s * P->r_s);
    for (int j = 0; j < kP2PPolyMax; ++j) k.c[j] = j < m ? (float)(coef[j] * inv8rs3) : 0.0f;
    k.ncoef = m > 0 ? m : 11;
    k.split = P->split;
    if (P->split == 1) k.c[0] = (float)(1.0 / P->r_cut);  // polynomial split: the FP32 kernel needs 1 / r_cut only
    k.two_over_rc2 = (float)(2.0 / (P->r_cut * P->r_cut));
    k.rc2 = (float)(P->r_cut * P->r_cut);
    return 0;
}

static const P2PConst64 &p2p_setup64(fmm_tree *t, const fmm_params *P)
{
    P2PLaw64 &w = t->law64;
    P2PConst64 &k = w.k;
    if (w.split == P->split && w.box == P->box && w.r_s == P->r_s && w.r_cut == P->r_cut) return k;
    law64_setup(P->r_s, P->r_cut, P->split, k);
    // the boxes are FP32 in the caller's units: tests only where these hold the boxes of leaves
    // down to 2^-21 of the box to P2PSink's margin
    const bool tests = P->box >= 0x1p-80 && P->box <= 0x1p100 && k.scale >= 0x1p-120 && k.scale <= 0x1p120;
    k.scale32 = tests ? (float)k.scale : 0.0f;
    k.cut = tests ? (float)(P->r_cut * k.scale) * 1.0001f : INFINITY;
    w.box = P->box;
    w.r_s = P->r_s;
    w.r_cut = P->r_cut;
    w.split = P->split;
    return k;
}

// The leaves' bounding boxes (they depend on the tree only).
int p2p_bbox(fmm_tree *t, const fmm_params *, hipStream_t st)
{
    if (t->nleaf == 0) return 0;
    if (int rc = grow(t->bbox, (size_t)t->ncell * 32)) return rc;
    k_leaf_bbox<<<(t->nleaf + 63) / 64, 64, 0, st>>>(ptr<Cell>(t->cells), ptr<int>(t->leaves), t->nleaf,
                                                    ptr<float4>(t->rel32), ptr<float4>(t->bbox));
    return hip_check(hipGetLastError(), "leaf boxes");
}

static void p2p_args(fmm_tree *t, P2PArgs &a)
{
    a.cells = ptr<Cell>(t->cells);
    a.leaves = ptr<int>(t->leaves);
    a.nleaf = t->nleaf;
    a.head = ptr<int>(t->lhead) + t->ncell;
    a.cnt = ptr<int>(t->lcnt) + t->ncell;
    a.items = ptr<uint32_t>(t->litems[1]);
    a.next = ptr<int>(t->lnext[1]);
    a.xs = ptr<double>(t->xs);
    a.ys = ptr<double>(t->ys);
    a.zs = ptr<double>(t->zs);
    a.ms = ptr<double>(t->ms);
    a.rel = ptr<float4>(t->rel32);
    a.box = t->box;
    a.nearf = ptr<double>(t->nearf);
    a.n = (int)t->n;
    a.slots = reinterpret_cast<unsigned long long *>(ptr<char>(t->counters) + kP2PByte);
    a.bbox = ptr<float4>(t->bbox);
    a.first = 0;
    a.err = nullptr;
    a.wide_cost = 1ll << 62;
    a.lcap = t->lcap[1];
    a.wide = ptr<int>(t->p2p_wide);
}

// Whether the fused persistent kernel serves these parameters: the FP32 plain form with
// the pair M2L kernel (orders 3..8) and a force law of degree 9 or 10, or the polynomial split.
bool fused_applies(const fmm_params *P)
{
    if (P->precision != 1 || P->learned || P->p < 3 || P->m2l_mfma == 2) return false;
    if (P->split == 1) return true;
    P2PConst k;
    return p2p_setup(P, k) == 0 && (k.ncoef == 10 || k.ncoef == 11);
}

template <bool POLY, int NPC, int P> static int launch_persist(fmm_tree *t, const P2PArgs &a, const P2PConst &k, Split sp,
                                                      int64_t np, int *queue, hipStream_t st)
{
    static int per_cu = 0, ncu = 0;
    if (per_cu == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_p2p_m2l_persist<POLY, NPC, P>, 64, 0) != hipSuccess ||
            per_cu <= 0)
            return set_error(FMM_ERR_HIP, "occupancy of the fused kernel");
    }
    const int64_t items = (int64_t)t->nleaf + (np + 63) / 64;
    const int64_t g = std::min<int64_t>(items, (int64_t)per_cu * ncu);
    if (g <= 0) return 0;
    k_p2p_m2l_persist<POLY, NPC, P><<<(unsigned)g, 64, 0, st>>>(a, k, ptr<int2>(t->m2l_pairs), np, ptr<float>(t->Mc),
                                                          ptr<float>(t->Lc), sp, ncoef(P), queue);
    return hip_check(hipGetLastError(), "fused p2p + m2l");
}

// P2P and M2L of a built tree (or forest) in one persistent launch on `st`.  The
// preparation (L zeroed, the M2L list flattened, the queue counter zeroed) is its own call
// so that stage timing can bracket the launch alone.
int p2p_m2l_fused_prepare(fmm_tree *t, const fmm_params *P, hipStream_t st)
{
    if (t->nleaf == 0) return 0;
    if (t->bbox.bytes < (size_t)t->ncell * 32) return set_error(FMM_ERR_STATE, "p2p: leaf boxes not computed");
    const int64_t np = t->n_m2l;
    if (int rc = zero_async(t->Lc.p, (size_t)t->ncell * ncoef(P->p) * sizeof(float), st)) return rc;
    if (np > 0)
        if (int rc = flatten_pairs(t, 0, np, st)) return rc;
    if (int rc = grow(t->m2l_ctr, 256)) return rc;
    return zero_async(ptr<int>(t->m2l_ctr) + 32, 4, st);
}

int p2p_m2l_fused_launch(fmm_tree *t, const fmm_params *P, hipStream_t st)
{
    if (t->nleaf == 0) return 0;
    P2PConst k;
    if (int rc = p2p_setup(P, k)) return rc;
    const int64_t np = t->n_m2l;
    int *queue = ptr<int>(t->m2l_ctr) + 32;
    P2PArgs a;
    p2p_args(t, a);
    const Split sp{P->split ? P->r_cut : P->r_s, P->split};
    if (P->split == 1) {
        switch (P->p) {
        case 3: return launch_persist<true, 11, 3>(t, a, k, sp, np, queue, st);
        case 4: return launch_persist<true, 11, 4>(t, a, k, sp, np, queue, st);
        case 5: return launch_persist<true, 11, 5>(t, a, k, sp, np, queue, st);
        case 6: return launch_persist<true, 11, 6>(t, a, k, sp, np, queue, st);
        case 7: return launch_persist<true, 11, 7>(t, a, k, sp, np, queue, st);
        case 8: return launch_persist<true, 11, 8>(t, a, k, sp, np, queue, st);
        }
    } else if (k.ncoef == 10) {
        switch (P->p) {
        case 3: return launch_persist<false, 10, 3>(t, a, k, sp, np, queue, st);
        case 4: return launch_persist<false, 10, 4>(t, a, k, sp, np, queue, st);
        case 5: return launch_persist<false, 10, 5>(t, a, k, sp, np, queue, st);
        case 6: return launch_persist<false, 10, 6>(t, a, k, sp, np, queue, st);
        case 7: return launch_persist<false, 10, 7>(t, a, k, sp, np, queue, st);
        case 8: return launch_persist<false, 10, 8>(t, a, k, sp, np, queue, st);
        }
    } else if (k.ncoef == 11) {
        switch (P->p) {
        case 3: return launch_persist<false, 11, 3>(t, a, k, sp, np, queue, st);
        case 4: return launch_persist<false, 11, 4>(t, a, k, sp, np, queue, st);
        case 5: return launch_persist<false, 11, 5>(t, a, k, sp, np, queue, st);
        case 6: return launch_persist<false, 11, 6>(t, a, k, sp, np, queue, st);
        case 7: return launch_persist<false, 11, 7>(t, a, k, sp, np, queue, st);
        case 8: return launch_persist<false, 11, 8>(t, a, k, sp, np, queue, st);
        }
    }
    return set_error(FMM_ERR_ARG, "fused kernel compiled for orders 3..8 and force laws of degree 9 or 10");
}

// One launch of k_p2p (count > 0: a wave per leaf) or k_p2p_wide (count = 0).
template <bool F64, bool POLY, int NPC, int CHUNK>
static void launch_one(const P2PLaw<F64> &k, const P2PArgs &a, int count, hipStream_t st)
{
    if (count > 0) k_p2p<F64, POLY, NPC, CHUNK><<<count, 64, 0, st>>>(a, k);
    else k_p2p_wide<F64, POLY, NPC, CHUNK><<<256, 64 * kWide, 0, st>>>(a, k);
}

template <int CHUNK>
static int launch_p2p(fmm_tree *t, const fmm_params *P, const P2PArgs &a, int count, hipStream_t st)
{
    if (!P->precision) {
        const P2PConst64 &k = p2p_setup64(t, P);
        if (k.ncoef == 1) launch_one<true, false, 1, CHUNK>(k, a, count, st);
        else if (k.ncoef == 19) launch_one<true, false, 19, CHUNK>(k, a, count, st);
        else if (k.ncoef == 22) launch_one<true, false, 22, CHUNK>(k, a, count, st);
        else launch_one<true, false, 0, CHUNK>(k, a, count, st);
        return hip_check(hipGetLastError(), "p2p");
    }
    P2PConst k;
    if (int rc = p2p_setup(P, k)) return rc;
    if (k.split == 1) launch_one<false, true, 11, CHUNK>(k, a, count, st);
    else if (k.ncoef == 10) launch_one<false, false, 10, CHUNK>(k, a, count, st);
    else if (k.ncoef == 11) launch_one<false, false, 11, CHUNK>(k, a, count, st);
    else if (k.ncoef == 15) launch_one<false, false, 15, CHUNK>(k, a, count, st);
    else return set_error(FMM_ERR_STATE, "p2p: no kernel for a force law of %d coefficients", k.ncoef);
    return hip_check(hipGetLastError(), "p2p");
}

int p2p_tile(const fmm_params *P) { return P->p2p_chunk == 16 || P->p2p_chunk == 64 ? P->p2p_chunk : kSinkChunk; }

static int launch_p2p(fmm_tree *t, const fmm_params *P, const P2PArgs &a, int count, hipStream_t st)
{
    if (P->p2p_chunk == 16) return launch_p2p<16>(t, P, a, count, st);
    if (P->p2p_chunk == 64) return launch_p2p<64>(t, P, a, count, st);
    return launch_p2p<kSinkChunk>(t, P, a, count, st);
}

int p2p_range(fmm_tree *t, const fmm_params *P, int first, int count, const int *err, hipStream_t st)
{
    if (count <= 0) return 0;
    if (first < 0 || count > t->nleaf - first) return set_error(FMM_ERR_STATE, "p2p: leaf range out of bounds");
    if (t->bbox.bytes < (size_t)t->ncell * 32) return set_error(FMM_ERR_STATE, "p2p: leaf boxes not computed");
    P2PArgs a;
    p2p_args(t, a);
    a.first = first;
    a.err = err;
    return launch_p2p(t, P, a, count, st);
}

// Where the line lies between one wave and a workgroup for a leaf, in p2p_cost: a leaf that
// would take a wave more than a quarter of the time the whole launch needs if evenly spread
// (over about four waves on each of the GPU's 1024 SIMDs) and at least four times the mean
// leaf.  One wave per leaf against this line (before, after): step of
// 300,007 particles 2.91 -> 1.79 ms (the costliest leaf alone took 2.2), 262,144 FP64 3.60 -> 2.57,
// 2M learned 8.4 -> 7.1, 2M plain 6.4 -> 6.1; 64-box forest and 16.7M box, whose launches are
// long beside any leaf, unchanged.
static long long wide_line(const fmm_tree *t)
{
    const long long even = t->n_p2p / 4096, mean = t->nleaf > 0 ? t->n_p2p / t->nleaf : 0;
    return std::max(std::max(even / 4, 4 * mean), 256ll);
}

// Selects the leaves for workgroups, on `st`.  *line receives the cost from which k_p2p leaves
// them out, or 2^62 if there are none.
int p2p_wide(fmm_tree *t, const fmm_params *P, hipStream_t st, long long *line)
{
    *line = 1ll << 62;
    // deterministic FP64 results are the same for every schedule: the one-wave order
    if (t->nleaf == 0 || (P->deterministic && !P->precision)) return 0;
    const long long cost = wide_line(t);
    if (t->p2p_max_cost < cost) return 0;  // no leaf is that costly
    if (int rc = grow(t->p2p_wide, ((size_t)t->nleaf + 1) * 4)) return rc;
    if (int rc = zero_async(t->p2p_wide.p, 4, st)) return rc;
    P2PArgs a;
    p2p_args(t, a);
    a.wide_cost = cost;
    const int nb = (t->nleaf + 63) / 64;
    if (P->p2p_chunk == 16) k_p2p_wide_select<16><<<nb, 64, 0, st>>>(a);
    else if (P->p2p_chunk == 64) k_p2p_wide_select<64><<<nb, 64, 0, st>>>(a);
    else k_p2p_wide_select<kSinkChunk><<<nb, 64, 0, st>>>(a);
    *line = cost;
    return hip_check(hipGetLastError(), "p2p selection");
}

int p2p_wide_launch(fmm_tree *t, const fmm_params *P, long long line, hipStream_t st)
{
    if (line >= 1ll << 62) return 0;
    P2PArgs a;
    p2p_args(t, a);
    a.wide_cost = line;
    return launch_p2p(t, P, a, 0, st);
}

int p2p(fmm_tree *t, const fmm_params *P, long long line, hipStream_t st)
{
    if (t->nleaf == 0) return 0;
    if (t->bbox.bytes < (size_t)t->ncell * 32) return set_error(FMM_ERR_STATE, "p2p: leaf boxes not computed");
    P2PArgs a;
    p2p_args(t, a);
    a.wide_cost = line;
    return launch_p2p(t, P, a, t->nleaf, st);
}

}  // namespace hfmm
