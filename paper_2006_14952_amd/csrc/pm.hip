// Long-range force by the particle-mesh method (Sec. 2.2): the Poisson Green function
// filtered by exp(-k^2 r_s^2), so that PM + the erfc-truncated short range sums to
// Newtonian gravity (the split of the force law g(r) of Sec. 2.2).
//
//   deposit -> rho(x);  FFT;  phi_k = -4 pi G rho_k exp(-k^2 r_s^2) / (k^2 W(k)^2);
//   a_k = -i k phi_k (three components);  inverse FFTs;  interpolation.
// The mass assignment is cloud-in-cell by default, or the higher-order triangular-shaped
// cloud (TSC) or piecewise cubic (PCS) B-spline schemes (fmm_params.pm_assign 3, 4);
// W(k) = prod_i sinc^p(k_i Delta / 2) is the window of the order-p scheme, divided out
// once for the deposit and once for the interpolation.  With the polynomial split the filter is the
// transform of its smoothing density 15/(8 pi r_c^3)(1 - r^2/r_c^2) (r < r_c):
// 15 (3 sin u - 3 u cos u - u^2 sin u) / u^5, u = k r_cut.  The k = 0 mode is dropped (mean density is
// cancelled by the expanding background).  FFTs are hipFFT (double precision).
#include <hipfft/hipfft.h>
#include <math.h>

#include <atomic>
#include <map>
#include <mutex>
#include <thread>
#include <type_traits>

#include "state.h"

namespace hfmm {
void clear_error();

struct PMPlan {
    int mesh = 0;
    hipfftHandle r2c = 0, c2r = 0;
    DevBuf rho, rhok, work, amesh;
    uint64_t behind = 0;  // number of the call whose launches may still use the buffers, 0: none
    hipEvent_t done = nullptr;  // their end
};

// Held while a call uses a plan on the host; on the device a call's launches wait for `done`.
static std::mutex g_pm_mu;
static std::map<int, PMPlan *> g_pm;  // one plan set per mesh size per process
// Caller-order particles brought into mesh order, for every mesh size, by the one call that holds
// g_order_busy.  The buffers (about 71 bytes a particle) are kept for the next call up to
// kOrderKeep particles, 2.7 GB, unless another buffer of the library needs the room first
// (release_idle).  Above, each call allocates and frees them: 40M particles on 256^3 9.3 ms, where
// kept buffers would make it 6.7 and the direct deposit takes 24.0.
static MortonSort g_order;
static std::atomic<bool> g_order_busy{false};
constexpr int kOrderKeep = 38000000;

static bool release_order()  // by the holder of g_order_busy; no launch uses the buffers
{
    MortonSort &s = g_order;
    bool any = false;
    for (DevBuf *b : {&s.keys[0], &s.keys[1], &s.idx[0], &s.idx[1], &s.xs, &s.ys, &s.zs, &s.ms, &s.tmp, &s.scan_tmp}) {
        any = any || b->p;
        release(*b);
    }
    return any;
}

bool release_idle()
{
    if (g_order_busy.exchange(true)) return false;
    const bool any = release_order();
    g_order_busy = false;
    return any;
}

// The order's buffers for one call (one at a time under g_pm_mu: only release_idle is waited for).
struct OrderUse {
    OrderUse()
    {
        while (g_order_busy.exchange(true)) std::this_thread::yield();
    }
    ~OrderUse() { g_order_busy = false; }
};

// The launches on st wait for those a call has left behind.
static int pm_wait(const PMPlan *pl, hipStream_t st)
{
    return pl->behind ? hip_check(hipStreamWaitEvent(st, pl->done, 0), "pm event wait") : 0;
}

static int pm_plan(int mesh, PMPlan **out)
{
    std::lock_guard<std::mutex> lk(g_pm_mu);
    auto it = g_pm.find(mesh);
    if (it != g_pm.end()) {
        *out = it->second;
        return 0;
    }
    PMPlan *p = new PMPlan();
    p->mesh = mesh;
    if (hipfftPlan3d(&p->r2c, mesh, mesh, mesh, HIPFFT_D2Z) != HIPFFT_SUCCESS ||
        hipfftPlan3d(&p->c2r, mesh, mesh, mesh, HIPFFT_Z2D) != HIPFFT_SUCCESS) {
        delete p;
        return set_error(FMM_ERR_HIP, "hipfftPlan3d(%d) failed", mesh);
    }
    size_t nr = (size_t)mesh * mesh * mesh, nc = (size_t)mesh * mesh * (mesh / 2 + 1);
    int rc = grow(p->rho, nr * 8) | grow(p->rhok, nc * 16) | grow(p->work, nc * 16) | grow(p->amesh, 3 * nr * 8);
    if (!rc) rc = hip_check(hipEventCreateWithFlags(&p->done, hipEventDisableTiming), "pm event");
    if (rc) {
        delete p;
        return rc;
    }
    g_pm[mesh] = p;
    *out = p;
    return 0;
}

// Mass-assignment weights of the B-spline schemes on the cell-centred mesh (node i at
// (i + 0.5) Delta): ORDER 2 cloud-in-cell, 3 triangular-shaped cloud, 4 piecewise cubic.
// Weights w[0 .. ORDER-1] of a particle's nodes along one axis; returns the first of them, which
// may lie outside [0, M).
template <int ORDER> __device__ __forceinline__ int assign_first(double x, double inv_d, double *w)
{
    const double g = x * inv_d - 0.5;
    double first;
    if constexpr (ORDER == 2) {
        const double f = floor(g), t = g - f;
        w[0] = 1.0 - t;
        w[1] = t;
        first = f;
    } else if constexpr (ORDER == 3) {
        const double c = floor(g + 0.5), dx = g - c;  // nearest node, dx in [-1/2, 1/2)
        w[0] = 0.5 * (0.5 - dx) * (0.5 - dx);
        w[1] = 0.75 - dx * dx;
        w[2] = 0.5 * (0.5 + dx) * (0.5 + dx);
        first = c - 1.0;
    } else {
        const double f = floor(g), t = g - f, t2 = t * t, t3 = t2 * t, u = 1.0 - t;
        w[0] = u * u * u / 6.0;
        w[1] = (4.0 - 6.0 * t2 + 3.0 * t3) / 6.0;
        w[2] = (1.0 + 3.0 * t + 3.0 * t2 - 3.0 * t3) / 6.0;
        w[3] = t3 / 6.0;
        first = f - 1.0;
    }
    return (int)first;
}

// The same with the first node wrapped: nodes i0 .. i0 + ORDER - 1 (mod M).
template <int ORDER> __device__ __forceinline__ void assign_weights(double x, double inv_d, int M, int &i0, double *w)
{
    const int i = assign_first<ORDER>(x, inv_d, w);
    i0 = ((i % M) + M) % M;
}

// Particle sources of the PM step: the caller's (n,3) positions and masses, or the
// octree's Morton-ordered SoA copies (wrapped), whose output rows are perm[p].  In Morton
// order neighbouring threads deposit into neighbouring mesh cells.
struct CallerOrder {
    const double *pos, *mass;
    __device__ double x(int p, int a) const { return pos[3 * (size_t)p + a]; }
    __device__ double m(int p) const { return mass[p]; }
    __device__ size_t row(int p) const { return 3 * (size_t)p; }
};
struct MortonOrder {
    const double *xs, *ys, *zs, *ms;
    const int *perm;
    __device__ double x(int p, int a) const { return a == 0 ? xs[p] : (a == 1 ? ys[p] : zs[p]); }
    __device__ double m(int p) const { return ms[p]; }
    __device__ size_t row(int p) const { return 3 * (size_t)perm[p]; }
};

template <class S, int ORDER>
__global__ void k_deposit(S src, int n, double box, int M, double inv_vol, double *__restrict__ rho)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    double inv_d = M / box;
    int i[3];
    double w[3][ORDER];
    for (int a = 0; a < 3; ++a) {
        double x = src.x(p, a);
        x -= box * floor(x / box);
        assign_weights<ORDER>(x, inv_d, M, i[a], w[a]);
    }
    double m = src.m(p) * inv_vol;
    for (int dx = 0; dx < ORDER; ++dx)
        for (int dy = 0; dy < ORDER; ++dy)
            for (int dz = 0; dz < ORDER; ++dz) {
                size_t idx = ((size_t)((i[0] + dx) % M) * M + (i[1] + dy) % M) * M + (i[2] + dz) % M;
                atomicAdd(&rho[idx], m * w[0][dx] * w[1][dy] * w[2][dz]);
            }
}

// Deposit of particles in Morton order.  A workgroup takes 4096 consecutive particles; those of
// one cube of 2^-levels the box (at most 19 - ORDER mesh cells wide) add into that cube's
// nodes in LDS, which then go to the mesh with one atomic per node: in clumps thousands of
// particles share a node, and same-address atomics on the mesh end one after the other
// (about 13 ns apart), while in random order every particle's eight atomics miss the caches.
// A workgroup whose particles lie in more than kDepositCubes cubes (a mesh much finer than the
// particles, whose nodes are hardly shared) adds straight to the mesh.
// 16.7M clustered particles on 256^3 (in this order): 6.27 -> 0.30 ms; the 2M box in tree order on
// 128^3: 1.81 -> 0.09 ms.
constexpr int kDepositThreads = 512, kDepositTile = 4096, kDepositSide = 20, kDepositPerCube = 128;
constexpr int kDepositCubes = kDepositTile / kDepositPerCube;
constexpr int kDepositPer = kDepositTile / kDepositThreads;

// Node index modulo M; nodes lie in [-2, M + 4] and M >= 8.
__device__ __forceinline__ int wrap_node(int i, int M) { return i < 0 ? i + M : i >= M ? i - M : i; }

// Where the cubes of a workgroup's particles begin (in no particular order); the number of
// cubes may exceed kDepositCubes, the places kept.
struct CubeHeads {
    int at[kDepositCubes], n;
};

__device__ __forceinline__ int find_cubes(CubeHeads &h, const uint64_t *__restrict__ keys, int base, int cnt, int sh)
{
    if (threadIdx.x == 0) h.n = 0;
    __syncthreads();
    for (int q = threadIdx.x; q < cnt; q += kDepositThreads)
        if (q == 0 || (keys[base + q] ^ keys[base + q - 1]) >> sh) {
            const int k = atomicAdd(&h.n, 1);
            if (k < kDepositCubes) h.at[k] = q;
        }
    __syncthreads();
    return h.n;
}

__device__ __forceinline__ int next_cube(const CubeHeads &h, int cubes, int beg, int cnt)
{
    int end = cnt;
    for (int k = 0; k < cubes; ++k)
        if (h.at[k] > beg && h.at[k] < end) end = h.at[k];
    return end;
}

// The nodes of the cube with Morton prefix `pre`: from its lowest corner's first to its highest
// corner's last, along each axis lo .. lo + len - 1 (unwrapped).
template <int ORDER> struct CubeNodes {
    int lo[3], len[3];
    __device__ __forceinline__ CubeNodes(uint64_t pre, int levels, double side, double inv_d)
    {
        for (int a = 0; a < 3; ++a) {
            int k = 0;
            for (int l = 0; l < levels; ++l) k |= (int)((pre >> (3 * l + 2 - a)) & 1) << l;
            double w[ORDER];
            lo[a] = assign_first<ORDER>(k * side, inv_d, w);
            len[a] = min(assign_first<ORDER>((k + 1) * side, inv_d, w) + ORDER - lo[a], kDepositSide);
        }
    }
    __device__ __forceinline__ int count() const { return len[0] * len[1] * len[2]; }
    // mesh index of node q of the cube
    __device__ __forceinline__ size_t mesh(int q, int M) const
    {
        const int iz = lo[2] + q % len[2], iy = lo[1] + q / len[2] % len[1], ix = lo[0] + q / (len[1] * len[2]);
        return ((size_t)wrap_node(ix, M) * M + wrap_node(iy, M)) * M + wrap_node(iz, M);
    }
    // cube index of a particle's first node, -1 if its nodes are not all among the cube's (a
    // particle on the cube's face, rounded to its other side)
    __device__ __forceinline__ int first(const int *i) const
    {
        for (int a = 0; a < 3; ++a)
            if (i[a] < lo[a] || i[a] + ORDER > lo[a] + len[a]) return -1;
        return ((i[0] - lo[0]) * len[1] + i[1] - lo[1]) * len[2] + i[2] - lo[2];
    }
};

template <int ORDER>
__global__ __launch_bounds__(kDepositThreads) void k_deposit_cubes(MortonOrder src, const uint64_t *__restrict__ keys,
                                                                   int levels, int n, int tile, double box, int M,
                                                                   double inv_vol, double *__restrict__ rho)
{
    __shared__ double acc[kDepositSide * kDepositSide * kDepositSide];
    __shared__ CubeHeads heads;
    const int base = blockIdx.x * tile, cnt = min(tile, n - base), sh = 63 - 3 * levels;
    const int cubes = find_cubes(heads, keys, base, cnt, sh);
    const double inv_d = M / box;
    auto direct = [&](const int *i, const double (*w)[ORDER], double m) __attribute__((always_inline)) {
        for (int dx = 0; dx < ORDER; ++dx)
            for (int dy = 0; dy < ORDER; ++dy)
                for (int dz = 0; dz < ORDER; ++dz) {
                    const int ix = wrap_node(i[0] + dx, M), iy = wrap_node(i[1] + dy, M), iz = wrap_node(i[2] + dz, M);
                    atomicAdd(&rho[((size_t)ix * M + iy) * M + iz], m * w[0][dx] * w[1][dy] * w[2][dz]);
                }
    };
    if (cubes > tile / kDepositPerCube) {
        for (int q = threadIdx.x; q < cnt; q += kDepositThreads) {
            const int p = base + q;
            int i[3];
            double w[3][ORDER];
            for (int a = 0; a < 3; ++a) i[a] = assign_first<ORDER>(src.x(p, a), inv_d, w[a]);
            direct(i, w, src.m(p) * inv_vol);
        }
        return;
    }
    const double side = ldexp(box, -levels);
    for (int beg = 0; beg < cnt;) {
        const int end = next_cube(heads, cubes, beg, cnt);
        const CubeNodes<ORDER> cube(keys[base + beg] >> sh, levels, side, inv_d);
        const int nnode = cube.count();
        for (int q = threadIdx.x; q < nnode; q += kDepositThreads) acc[q] = 0.0;
        __syncthreads();
        for (int q = beg + threadIdx.x; q < end; q += kDepositThreads) {
            const int p = base + q;
            int i[3];
            double w[3][ORDER];
            for (int a = 0; a < 3; ++a) i[a] = assign_first<ORDER>(src.x(p, a), inv_d, w[a]);
            const double m = src.m(p) * inv_vol;
            const int o = cube.first(i);
            if (o < 0) {
                direct(i, w, m);
                continue;
            }
            for (int dx = 0; dx < ORDER; ++dx)
                for (int dy = 0; dy < ORDER; ++dy)
                    for (int dz = 0; dz < ORDER; ++dz)
                        atomicAdd(&acc[o + (dx * cube.len[1] + dy) * cube.len[2] + dz], m * w[0][dx] * w[1][dy] * w[2][dz]);
        }
        __syncthreads();
        for (int q = threadIdx.x; q < nnode; q += kDepositThreads)
            if (acc[q] != 0.0) atomicAdd(&rho[cube.mesh(q, M)], acc[q]);
        __syncthreads();
        beg = end;
    }
}

// Deterministic deposit (fmm_params.deterministic): every contribution m w / d^3 is rounded
// to an integer multiple of 2^-e and summed in 64-bit integers, whose sums do not depend on
// the order of the atomics.  e is the largest exponent with n max|m| / d^3 2^e < 2^62, so no
// partial sum overflows; a contribution's rounding is at most 2^-(e+1), below 1e-15 of the
// total |mass| / d^3 for any n up to 2^30.
template <class S> __global__ __launch_bounds__(256) void k_mass_absmax(S src, int n, unsigned long long *mx)
{
    __shared__ unsigned long long w[256];
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    // |m| >= 0: the order of the bit patterns is the order of the values
    w[threadIdx.x] = p < n ? (unsigned long long)__double_as_longlong(fabs(src.m(p))) : 0ull;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) w[threadIdx.x] = max(w[threadIdx.x], w[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0 && w[0]) atomicMax(mx, w[0]);
}

__device__ __forceinline__ int fixed_exponent(const unsigned long long *mx, int n, double inv_vol)
{
    const double bound = (double)n * __longlong_as_double((long long)*mx) * inv_vol;
    return bound > 0.0 ? 61 - ilogb(bound) : 0;
}

template <class S, int ORDER>
__global__ void k_deposit_fixed(S src, int n, double box, int M, double inv_vol, const unsigned long long *__restrict__ mx,
                                unsigned long long *__restrict__ rho)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int e = fixed_exponent(mx, n, inv_vol);
    double inv_d = M / box;
    int i[3];
    double w[3][ORDER];
    for (int a = 0; a < 3; ++a) {
        double x = src.x(p, a);
        x -= box * floor(x / box);
        assign_weights<ORDER>(x, inv_d, M, i[a], w[a]);
    }
    double m = src.m(p) * inv_vol;
    for (int dx = 0; dx < ORDER; ++dx)
        for (int dy = 0; dy < ORDER; ++dy)
            for (int dz = 0; dz < ORDER; ++dz) {
                size_t idx = ((size_t)((i[0] + dx) % M) * M + (i[1] + dy) % M) * M + (i[2] + dz) % M;
                const long long q = llrint(ldexp(m * w[0][dx] * w[1][dy] * w[2][dz], e));
                atomicAdd(&rho[idx], (unsigned long long)q);
            }
}

// The integer mesh back to FP64, in place.
__global__ void k_fixed_to_double(unsigned long long *__restrict__ rho, size_t nr, const unsigned long long *__restrict__ mx,
                                  int n, double inv_vol)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nr) return;
    const int e = fixed_exponent(mx, n, inv_vol);
    const double v = ldexp((double)(long long)rho[i], -e);
    reinterpret_cast<double *>(rho)[i] = v;
}

__device__ __forceinline__ double sinc(double x) { return fabs(x) < 1e-8 ? 1.0 : sin(x) / x; }

// long-range filter at |k|^2 = k2: Gaussian split exp(-k^2 r_s^2); polynomial split the
// transform above (its series below u = 0.1, where the closed form cancels)
__device__ __forceinline__ double lr_window(double k2, double rs, int split, double rcut)
{
    if (split != 1) return exp(-k2 * rs * rs);
    const double u = sqrt(k2) * rcut, u2 = u * u;
    if (u < 0.1) return 1.0 - u2 / 14.0 + u2 * u2 / 504.0 - u2 * u2 * u2 / 33264.0;
    const double s = sin(u), c = cos(u);
    return 15.0 * (3.0 * s - 3.0 * u * c - u2 * s) / (u2 * u2 * u);
}

// a_k component `axis` from rho_k; includes the 1/M^3 of the inverse transform
__global__ void k_green_grad(const hipfftDoubleComplex *__restrict__ rhok, hipfftDoubleComplex *__restrict__ out,
                             int M, double box, double rs, int split, double rcut, double G, int axis, int order)
{
    int Mh = M / 2 + 1;
    size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t nc = (size_t)M * M * Mh;
    if (t >= nc) return;
    int kz = (int)(t % Mh), ky = (int)((t / Mh) % M), kx = (int)(t / ((size_t)Mh * M));
    int nx = kx <= M / 2 ? kx : kx - M, ny = ky <= M / 2 ? ky : ky - M, nz = kz;
    double twopi_L = 2.0 * M_PI / box, d = box / M;
    double k0 = nx * twopi_L, k1 = ny * twopi_L, k2 = nz * twopi_L;
    double k2s = k0 * k0 + k1 * k1 + k2 * k2;
    hipfftDoubleComplex r = rhok[t], o;
    if (k2s == 0.0 || (M % 2 == 0 && (nx == M / 2 || ny == M / 2 || nz == M / 2))) {
        o.x = 0; o.y = 0;  // k = 0 and the unpaired Nyquist planes carry no gradient
        out[t] = o;
        return;
    }
    const double s1 = sinc(0.5 * k0 * d) * sinc(0.5 * k1 * d) * sinc(0.5 * k2 * d);
    double W = s1;  // the assignment window: sinc^order per axis
    for (int o = 1; o < order; ++o) W *= s1;
    double phi = -4.0 * M_PI * G * lr_window(k2s, rs, split, rcut) / (k2s * W * W);
    double ka = axis == 0 ? k0 : (axis == 1 ? k1 : k2);
    double s = phi * ka / ((double)M * M * M);  // a_k = -i k phi_k
    o.x = s * r.y;
    o.y = -s * r.x;
    out[t] = o;
}

template <class S, int ORDER>
__global__ void k_interp(S src, int n, double box, int M, const double *__restrict__ am, double *__restrict__ acc)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    double inv_d = M / box;
    int i[3];
    double w[3][ORDER];
    for (int a = 0; a < 3; ++a) {
        double x = src.x(p, a);
        x -= box * floor(x / box);
        assign_weights<ORDER>(x, inv_d, M, i[a], w[a]);
    }
    size_t nr = (size_t)M * M * M;
    double g[3] = {0, 0, 0};
    for (int dx = 0; dx < ORDER; ++dx)
        for (int dy = 0; dy < ORDER; ++dy)
            for (int dz = 0; dz < ORDER; ++dz) {
                const double wt = w[0][dx] * w[1][dy] * w[2][dz];
                size_t idx = ((size_t)((i[0] + dx) % M) * M + (i[1] + dy) % M) * M + (i[2] + dz) % M;
                for (int a = 0; a < 3; ++a) g[a] += wt * am[a * nr + idx];
            }
    const size_t o = src.row(p);
    for (int a = 0; a < 3; ++a) acc[o + a] = g[a];
}

// Interpolation to particles in Morton order: as k_deposit_cubes, with a cube's nodes of one
// component at a time in LDS (read once for all its particles, coalesced) and the particles'
// three sums in registers.  For particles ordered to the cubes only (within one they are in the
// caller's order), from 2^21 of them and two cells a particle on, and 8 or 27 nodes a particle:
// 16.7M on 256^3 1.37 -> 1.09 ms, 4M on 160^3 with 27 nodes 1.43 -> 1.20 in all; below, and in tree
// order (2M on 128^3 0.14 against 0.12 ms), the plain gather is as fast, and 64 nodes a particle
// leave this form too few registers.
template <int ORDER>
__global__ __launch_bounds__(kDepositThreads) void k_interp_cubes(MortonOrder src, const uint64_t *__restrict__ keys,
                                                                  int levels, int n, double box, int M,
                                                                  const double *__restrict__ am, double *__restrict__ acc)
{
    __shared__ double node[kDepositSide * kDepositSide * kDepositSide];
    __shared__ CubeHeads heads;
    const int base = blockIdx.x * kDepositTile, cnt = min(kDepositTile, n - base), sh = 63 - 3 * levels;
    const int cubes = find_cubes(heads, keys, base, cnt, sh);
    const double inv_d = M / box, side = ldexp(box, -levels);
    const size_t nr = (size_t)M * M * M;
    auto direct = [&](const int *i, const double (*w)[ORDER], int a) __attribute__((always_inline)) {
        double g = 0;
        for (int dx = 0; dx < ORDER; ++dx)
            for (int dy = 0; dy < ORDER; ++dy)
                for (int dz = 0; dz < ORDER; ++dz) {
                    const int ix = wrap_node(i[0] + dx, M), iy = wrap_node(i[1] + dy, M), iz = wrap_node(i[2] + dz, M);
                    g += w[0][dx] * w[1][dy] * w[2][dz] * am[a * nr + ((size_t)ix * M + iy) * M + iz];
                }
        return g;
    };
    if (cubes > kDepositCubes) {
        for (int q = threadIdx.x; q < cnt; q += kDepositThreads) {
            const int p = base + q;
            int i[3];
            double w[3][ORDER];
            for (int a = 0; a < 3; ++a) i[a] = assign_first<ORDER>(src.x(p, a), inv_d, w[a]);
            const size_t o = src.row(p);
            for (int a = 0; a < 3; ++a) acc[o + a] = direct(i, w, a);
        }
        return;
    }
    for (int beg = 0; beg < cnt;) {
        const int end = next_cube(heads, cubes, beg, cnt);
        const CubeNodes<ORDER> cube(keys[base + beg] >> sh, levels, side, inv_d);
        const int nnode = cube.count();
        double g[kDepositPer][3];
        unsigned outside = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            for (int q = threadIdx.x; q < nnode; q += kDepositThreads) node[q] = am[a * nr + cube.mesh(q, M)];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kDepositPer; ++r) {
                const int q = beg + threadIdx.x + r * kDepositThreads, p = base + q;
                g[r][a] = 0.0;
                if (q >= end) continue;
                int i[3];
                double w[3][ORDER];
                for (int b = 0; b < 3; ++b) i[b] = assign_first<ORDER>(src.x(p, b), inv_d, w[b]);
                const int o = cube.first(i);
                if (o < 0) {
                    outside |= 1u << r;
                    continue;
                }
                for (int dx = 0; dx < ORDER; ++dx)
                    for (int dy = 0; dy < ORDER; ++dy)
                        for (int dz = 0; dz < ORDER; ++dz)
                            g[r][a] += w[0][dx] * w[1][dy] * w[2][dz] * node[o + (dx * cube.len[1] + dy) * cube.len[2] + dz];
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < kDepositPer; ++r) {
            const int q = beg + threadIdx.x + r * kDepositThreads;
            if (q >= end) continue;
            const size_t o = src.row(base + q);
            for (int a = 0; a < 3; ++a) acc[o + a] = g[r][a];
        }
        for (int r = 0; outside >> r; ++r) {
            if (!(outside >> r & 1)) continue;
            const int p = base + beg + threadIdx.x + r * kDepositThreads;
            int i[3];
            double w[3][ORDER];
            for (int b = 0; b < 3; ++b) i[b] = assign_first<ORDER>(src.x(p, b), inv_d, w[b]);
            const size_t o = src.row(p);
            for (int a = 0; a < 3; ++a) acc[o + a] = direct(i, w, a);
        }
        beg = end;
    }
}

__global__ void k_add3(double *__restrict__ acc, const double *__restrict__ other, size_t n3)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n3) acc[i] += other[i];
}

// out[0]: a position is not finite; out[1]: particles in the mesh cell of the one before them;
// out[2] (LAG): particles in the mesh cell of the one 64 places before.
constexpr int kRunLag = 64;

__device__ __forceinline__ bool same_cell(const double *__restrict__ pos, int i, int j, double inv_d)
{
    bool eq = true;
    for (int a = 0; a < 3; ++a)
        eq = eq && floor(pos[3 * (size_t)i + a] * inv_d) == floor(pos[3 * (size_t)j + a] * inv_d);
    return eq;
}

template <bool LAG>
__global__ __launch_bounds__(256) void k_check_positions(const double *__restrict__ pos, int n, double inv_d,
                                                         int *__restrict__ out)
{
    __shared__ int same[2];
    if (threadIdx.x < 2) same[threadIdx.x] = 0;
    __syncthreads();
    int mine = 0, far = 0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        for (int a = 0; a < 3; ++a)
            if (!isfinite(pos[3 * (size_t)i + a])) out[0] = 1;
        if (i > 0) mine += same_cell(pos, i, i - 1, inv_d);
        if (LAG && i >= kRunLag) far += same_cell(pos, i, i - kRunLag, inv_d);
    }
    for (int o = 32; o > 0; o >>= 1) {
        mine += __shfl_xor(mine, o, 64);
        if (LAG) far += __shfl_xor(far, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        if (mine) atomicAdd(&same[0], mine);
        if (far) atomicAdd(&same[1], far);
    }
    __syncthreads();
    if (threadIdx.x < 2 && same[threadIdx.x]) atomicAdd(&out[1 + threadIdx.x], same[threadIdx.x]);
}

// Whether to bring n caller-order particles into mesh order: always if enough of them share the
// mesh's nodes (dense), else if many lie in the cell of the one before (kSameMin).  Two things
// make the direct deposit slow: particles of a clump that follow each other in the caller's
// arrays and queue on the same nodes (some 10 ns each, against 0.1 to 0.2 ms for the order), and
// mesh nodes that miss the caches.  Measured, ms direct / ordered: clustered 65,536 on 32^3
// 0.34 / 0.15, 100,000 on 64^3 0.40 / 0.20; uniform 500,000 on 80^3 0.41 / 0.33, 1,048,576 on
// 100^3 0.81 / 0.44, but 1,000,000 on 250^3, whose nodes hardly two particles share,
// 1.92 / 2.06.  Particles that come in mesh order follow each other in their cells although
// nothing queues: there the order pays from some 100,000 of them on (uniform ones so sorted, on
// 16^3: 65,536 0.114 / 0.123, 100,000 0.149 / 0.135), and below if cells hold so many that the
// one 64 places before is still in them (kFarMin: clustered 30,000 on 16^3 0.37 / 0.16).
static bool dense(int n, int mesh) { return n >= 1 << 19 && 8.0 * n >= (double)mesh * mesh * mesh; }
constexpr int kSameMin = 1 << 14, kFarMin = 2000, kManyMin = 100000;

// Morton levels at which a cube is at most 19 - order mesh cells wide (k_deposit_cubes).
static int cube_levels(int mesh, int order)
{
    int l = 0;
    while (mesh > (19 - order) << l) ++l;
    return l;
}

// Particles per workgroup of k_deposit_cubes: fewer where 4,096 would leave the chip idle (64
// nodes a particle on 64^3, clumps in mesh order: 65,536 particles in tiles of 4,096 1.75 ms, of
// 512 0.45; the direct deposit 0.70).  But where a cube takes several tiles, each sends all of the
// cube's nodes to the mesh, so a tile then keeps several contributions a node (8 nodes a particle
// on 16^3, one cube, 300,000 uniform: tiles of 4,096 0.215 ms, of 512 0.233).
static int deposit_tile(int n, int levels, int order)
{
    const int cube = n >> 3 * levels, several = order == 4 ? 512 : order == 3 ? 1024 : kDepositTile;
    const int least = cube < several ? cube : several;
    int t = kDepositTile;
    while (t > kDepositThreads && n / t < 512 && t / 2 >= least) t /= 2;
    return t;
}

// keys: the Morton keys of src's particles, in order by their first 3 cube_levels bits
// (full_order: by far more than a mesh cell's), or nullptr (any order).
template <class S>
static int pm_run(PMPlan *pl, const fmm_params *P, int mesh, int n, S src, const uint64_t *keys, bool full_order,
                  double *acc, hipStream_t st)
{
    size_t nr = (size_t)mesh * mesh * mesh, nc = (size_t)mesh * mesh * (mesh / 2 + 1);
    if (int rc = hip_check(hipMemsetAsync(pl->rho.p, 0, nr * 8, st), "pm mesh")) return rc;
    double d = P->box / mesh;
    const int order = P->pm_assign == 0 ? 2 : P->pm_assign;
    const unsigned nb = (unsigned)((n + 255) / 256);
    const double inv_vol = 1.0 / (d * d * d);
    if (P->deterministic) {
        unsigned long long *mx = ptr<unsigned long long>(pl->amesh);  // the output mesh is not yet in use
        unsigned long long *irho = ptr<unsigned long long>(pl->rho);
        if (int rc = hip_check(hipMemsetAsync(mx, 0, 8, st), "pm mass bound")) return rc;
        k_mass_absmax<S><<<nb, 256, 0, st>>>(src, n, mx);
        if (order == 3) k_deposit_fixed<S, 3><<<nb, 256, 0, st>>>(src, n, P->box, mesh, inv_vol, mx, irho);
        else if (order == 4) k_deposit_fixed<S, 4><<<nb, 256, 0, st>>>(src, n, P->box, mesh, inv_vol, mx, irho);
        else k_deposit_fixed<S, 2><<<nb, 256, 0, st>>>(src, n, P->box, mesh, inv_vol, mx, irho);
        k_fixed_to_double<<<(unsigned)((nr + 255) / 256), 256, 0, st>>>(irho, nr, mx, n, inv_vol);
    } else if (keys) {
        if constexpr (std::is_same<S, MortonOrder>::value) {
            const int lv = cube_levels(mesh, order), tile = deposit_tile(n, lv, order);
            const unsigned g = (unsigned)((n + tile - 1) / tile);
            double *rho = ptr<double>(pl->rho);
            if (order == 3) k_deposit_cubes<3><<<g, kDepositThreads, 0, st>>>(src, keys, lv, n, tile, P->box, mesh, inv_vol, rho);
            else if (order == 4) k_deposit_cubes<4><<<g, kDepositThreads, 0, st>>>(src, keys, lv, n, tile, P->box, mesh, inv_vol, rho);
            else k_deposit_cubes<2><<<g, kDepositThreads, 0, st>>>(src, keys, lv, n, tile, P->box, mesh, inv_vol, rho);
        }
    } else if (order == 3) {
        k_deposit<S, 3><<<nb, 256, 0, st>>>(src, n, P->box, mesh, inv_vol, ptr<double>(pl->rho));
    } else if (order == 4) {
        k_deposit<S, 4><<<nb, 256, 0, st>>>(src, n, P->box, mesh, inv_vol, ptr<double>(pl->rho));
    } else {
        k_deposit<S, 2><<<nb, 256, 0, st>>>(src, n, P->box, mesh, inv_vol, ptr<double>(pl->rho));
    }
    if (hipfftSetStream(pl->r2c, st) != HIPFFT_SUCCESS || hipfftSetStream(pl->c2r, st) != HIPFFT_SUCCESS)
        return set_error(FMM_ERR_HIP, "hipfftSetStream");
    if (hipfftExecD2Z(pl->r2c, ptr<double>(pl->rho), ptr<hipfftDoubleComplex>(pl->rhok)) != HIPFFT_SUCCESS)
        return set_error(FMM_ERR_HIP, "hipfftExecD2Z");
    for (int axis = 0; axis < 3; ++axis) {
        k_green_grad<<<(unsigned)((nc + 255) / 256), 256, 0, st>>>(ptr<hipfftDoubleComplex>(pl->rhok),
                                                                  ptr<hipfftDoubleComplex>(pl->work), mesh, P->box,
                                                                  P->r_s, P->split, P->r_cut, P->G, axis, order);
        if (hipfftExecZ2D(pl->c2r, ptr<hipfftDoubleComplex>(pl->work), ptr<double>(pl->amesh) + axis * nr) !=
            HIPFFT_SUCCESS)
            return set_error(FMM_ERR_HIP, "hipfftExecZ2D");
    }
    bool cubed = false;
    if constexpr (std::is_same<S, MortonOrder>::value) {
        cubed = keys && !full_order && order <= 3 && n >= 1 << 21 && 2 * (size_t)n >= nr;
        const unsigned g = (unsigned)((n + kDepositTile - 1) / kDepositTile);
        const int lv = cube_levels(mesh, order);
        const double *am = ptr<double>(pl->amesh);
        if (cubed && order == 3) k_interp_cubes<3><<<g, kDepositThreads, 0, st>>>(src, keys, lv, n, P->box, mesh, am, acc);
        else if (cubed) k_interp_cubes<2><<<g, kDepositThreads, 0, st>>>(src, keys, lv, n, P->box, mesh, am, acc);
    }
    if (cubed) {}
    else if (order == 3) k_interp<S, 3><<<nb, 256, 0, st>>>(src, n, P->box, mesh, ptr<double>(pl->amesh), acc);
    else if (order == 4) k_interp<S, 4><<<nb, 256, 0, st>>>(src, n, P->box, mesh, ptr<double>(pl->amesh), acc);
    else k_interp<S, 2><<<nb, 256, 0, st>>>(src, n, P->box, mesh, ptr<double>(pl->amesh), acc);
    return hip_check(hipGetLastError(), "pm");
}

int pm_forces(const fmm_params *P, int mesh, int64_t n64, const double *pos, const double *mass, double *acc,
              hipStream_t st)
{
    if (mesh < 8 || mesh > 1024) return set_error(FMM_ERR_ARG, "mesh must be in [8, 1024]");
    if (n64 < 0 || n64 > ((int64_t)1 << 30)) return set_error(FMM_ERR_ARG, "n out of range");
    const int n = (int)n64;
    if (n == 0) return 0;
    PMPlan *pl;
    if (int rc = pm_plan(mesh, &pl)) return rc;
    std::lock_guard<std::mutex> lk(g_pm_mu);  // plans and their buffers are shared per mesh size
    if (int rc = pm_wait(pl, st)) return rc;
    int *check = ptr<int>(pl->amesh), found[4] = {0, 0, 0, 0};  // scratch in the (not yet used) output mesh
    if (int rc = hip_check(hipMemsetAsync(check, 0, sizeof(found), st), "pm check")) return rc;
    auto read_check = [&]() -> int {
        if (hipMemcpyAsync(found, check, sizeof(found), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return set_error(FMM_ERR_HIP, "pm sync");
        return found[0] ? set_error(FMM_ERR_NAN, "non-finite particle position") : 0;
    };
    auto check_all = [&]() -> int {
        const int nb = (n + 255) / 256;
        const auto kernel = n < kManyMin ? k_check_positions<true> : k_check_positions<false>;
        kernel<<<nb < 2048 ? nb : 2048, 256, 0, st>>>(pos, n, mesh / P->box, check);
        return read_check();
    };
    const bool sure = !P->deterministic && dense(n, mesh);  // the keys' pass finds non-finite positions too
    if (!sure)
        if (int rc = check_all()) return rc;
    const bool runs = found[1] >= kSameMin && (n >= kManyMin || found[2] >= kFarMin);
    if (sure || (!P->deterministic && runs)) {
        const int order = P->pm_assign == 0 ? 2 : P->pm_assign;
        const OrderUse use;
        MortonSort &s = g_order;
        int rc = morton_order(s, n, P->box, pos, mass, cube_levels(mesh, order), check, st);
        const bool no_room = rc == FMM_ERR_NOMEM;
        if (rc == 0 && (!sure || (rc = read_check()) == 0))
            rc = pm_run(pl, P, mesh, n,
                        MortonOrder{ptr<double>(s.xs), ptr<double>(s.ys), ptr<double>(s.zs), ptr<double>(s.ms),
                                    ptr<int>(s.idx[s.sorted])},
                        ptr<uint64_t>(s.keys[s.sorted]), false, acc, st);
        if (!no_room) {
            const int rc_sync = hip_check(hipStreamSynchronize(st), "pm");  // the buffers are the next call's
            if (n > kOrderKeep) (void)release_order();
            return rc ? rc : rc_sync;
        }
        clear_error();  // no room for the order: the particles as they come
        (void)release_order();
        if (sure)
            if (int rc2 = check_all()) return rc2;
    }
    if (int rc = pm_run(pl, P, mesh, n, CallerOrder{pos, mass}, nullptr, false, acc, st)) return rc;
    return hip_check(hipStreamSynchronize(st), "pm");
}

// PM on the particles of a built tree (Morton order, already wrapped and checked), enqueued on
// st.  The plan's buffers are the next call's once `done` has passed, so the host lock covers
// the launches only: hybrid steps of several threads share the mesh part one after the other,
// and nothing else.  *call receives the call's number for pm_tree_done (0: nothing launched).
int pm_forces_tree(const fmm_params *P, int mesh, fmm_tree *t, double *acc, hipStream_t st, uint64_t *call)
{
    static uint64_t calls = 0;  // under g_pm_mu
    *call = 0;
    if (mesh < 8 || mesh > 1024) return set_error(FMM_ERR_ARG, "mesh must be in [8, 1024]");
    if (t->n == 0) return 0;
    PMPlan *pl;
    if (int rc = pm_plan(mesh, &pl)) return rc;
    std::lock_guard<std::mutex> lk(g_pm_mu);
    if (int rc = pm_wait(pl, st)) return rc;
    const int rc = pm_run(pl, P, mesh, (int)t->n,
                          MortonOrder{ptr<double>(t->xs), ptr<double>(t->ys), ptr<double>(t->zs), ptr<double>(t->ms),
                                      ptr<int>(t->perm)},
                          ptr<uint64_t>(t->keys[t->sorted]), true, acc, st);
    *call = pl->behind = ++calls;  // after an error too
    const int rc_done = hip_check(hipEventRecord(pl->done, st), "pm event");
    return rc ? rc : rc_done;
}

// At a hybrid step's end, when its mesh part has long ended: the next call need not wait for it
// on the device (a wait for an event of another stream costs some 10 us).
int pm_tree_done(int mesh, uint64_t call)
{
    PMPlan *pl;
    if (int rc = pm_plan(mesh, &pl)) return rc;
    {
        std::lock_guard<std::mutex> lk(g_pm_mu);
        if (pl->behind != call) return 0;  // a later call waits for this one
    }
    if (int rc = hip_check(hipEventSynchronize(pl->done), "pm")) return rc;
    std::lock_guard<std::mutex> lk(g_pm_mu);
    if (pl->behind == call) pl->behind = 0;
    return 0;
}

int add_into(double *acc, const double *other, int64_t n3, hipStream_t st)
{
    if (n3 <= 0) return 0;
    k_add3<<<(unsigned)((n3 + 255) / 256), 256, 0, st>>>(acc, other, (size_t)n3);
    return hip_check(hipGetLastError(), "add");
}

}  // namespace hfmm
