// ttm_compact.hip -- the compact sixth-order first derivative of Sec. 4.2,
// Eq. (cfds), applied along one mode of a periodic 3-way field without forming
// D = A_c^-1 B_c.  Two solvers of the cyclic tridiagonal system:
//
// Single pass (fibers of any length, |alpha| up to about 0.42 in float64 and
// 0.48 in float32): the circulant factorization of A_c below turns the solve
// into two first-order recursions that forget their start after K <= 64
// points, so each point is read once and written once (the algorithmic two
// transfers).
//
// Exact sweeps (alpha nearer to 1/2): the five-point right-hand side is built on
// the fly and fused with the forward pass of a cyclic tridiagonal solve
// (Sec. 2.1, the periodic Thomas algorithm, here as a Sherman-Morrison
// correction of one tridiagonal solve); the correction's scalar is
// accumulated during the forward pass, so one backward pass finishes the
// solve.  Splitting (gamma = -1): A_c = T + p q^T, T tridiagonal with alpha
// beside the diagonal and diagonal 1 except T_00 = 1 - gamma, T_{n-1,n-1} =
// 1 - alpha^2 / gamma; p = (gamma, 0, .., 0, alpha), q = (1, 0, .., 0, alpha /
// gamma).  With T y = d and T z = p the solution is x = y - [q.y / (1 + q.z)]
// z.  The fiber-independent data -- inv_j and cp_j of T's forward pass, z, and
// weights w_j with y_0 = sum_j w_j y'_j (y' the forward-pass values) -- come
// from one device thread in double precision before the sweep.  The forward
// pass stores y' into Y and the backward pass turns it into the solution in
// place: four transfers per point.
//
// Layout: one lane per fiber for modes 1 and 2, as the paper gives each GPU
// thread one line of a group of SZ lines (Sec. 4.1): row-major X makes those
// fibers interleaved already (lane f and f+1 read neighbouring addresses at
// every step).  Mode-3 fibers are contiguous rows, moved through LDS tiles.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "ttm_device.hpp"
#include "ttm_host.hpp"

namespace ttm {

namespace {

constexpr int64_t COMPACT_PREP_LDS_MAX = 8192;   // fibers up to this length keep the prep in LDS

struct CompactArgs {
    int64_t n, stride, nfib, i3;   // fiber length and element stride; fibers; I3 (mode 2 mapping)
    int64_t s12;                   // I2 * I3
    int mode;
    double ca, cb, alpha;          // a / (2h), b / (4h), alpha
};

// ws layout (elements of T): inv[n] | cp[n] | w[n] | z[n] | k, alpha/gamma.
// One thread runs the forward pass of T (and of T z = p) in double, keeping
// z' and cp in LDS when they fit (dynamic LDS of 16 n bytes, else read back
// from the workspace), then z's backward pass.
template <typename T>
__global__ void __launch_bounds__(64) k_compact_prep(int64_t n, double alpha, T *ws) {
    extern __shared__ __align__(16) unsigned char smem_prep[];
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const double gamma = -1.0;
    T *inv = ws, *cp = ws + n, *w = ws + 2 * n, *z = ws + 3 * n;
    const bool lds = n <= COMPACT_PREP_LDS_MAX;
    double *zl = reinterpret_cast<double *>(smem_prep), *cl = zl + (lds ? n : 0);
    double cprev = 0.0, zf = 0.0, wj = 1.0;
    for (int64_t j = 0; j < n; ++j) {
        const double dj = (j == 0) ? 1.0 - gamma : (j == n - 1 ? 1.0 - alpha * alpha / gamma : 1.0);
        const double iv = 1.0 / (dj - (j > 0 ? alpha * cprev : 0.0));
        const double pj = (j == 0) ? gamma : (j == n - 1 ? alpha : 0.0);
        zf = (pj - (j > 0 ? alpha * zf : 0.0)) * iv;
        if (j > 0) wj = -cprev * wj;
        cprev = alpha * iv;
        inv[j] = T(iv);
        cp[j] = T(cprev);
        w[j] = T(wj);
        if (lds) { zl[j] = zf; cl[j] = cprev; }
        else z[j] = T(zf);                // forward value, replaced below
    }
    const double zlast = zf;              // z_{n-1} = z'_{n-1}
    double zn = zlast;
    z[n - 1] = T(zn);
    for (int64_t j = n - 2; j >= 0; --j) {
        zn = (lds ? zl[j] - cl[j] * zn : double(z[j]) - double(cp[j]) * zn);
        z[j] = T(zn);
    }
    ws[4 * n] = T(1.0 / (1.0 + zn + (alpha / gamma) * zlast));   // zn = z_0 here
    ws[4 * n + 1] = T(alpha / gamma);
}

template <typename T>
__global__ void __launch_bounds__(256) k_compact(const CompactArgs a, const T *__restrict__ X, T *__restrict__ Y,
                                                 const T *__restrict__ ws) {
    for (int64_t f = int64_t(blockIdx.x) * 256 + threadIdx.x; f < a.nfib; f += int64_t(gridDim.x) * 256) {
    int64_t base;
    if (a.mode == 1) base = f;
    else if (a.mode == 2) base = (f / a.i3) * a.s12 + f % a.i3;
    else base = f * a.n;
    const int64_t n = a.n, s = a.stride;
    const T *u = X + base;
    T *y = Y + base;
    const T *inv = ws, *cp = ws + n, *w = ws + 2 * n, *z = ws + 3 * n;
    const T kk = ws[4 * n], ag = ws[4 * n + 1];
    const T ca = T(a.ca), cb = T(a.cb), alpha = T(a.alpha);

    // forward: d_j from the window u_{j-2} .. u_{j+2} (indices mod n), then
    // y'_j = (d_j - alpha y'_{j-1}) inv_j, stored in Y; q.y accumulates
    const T u0 = u[0], u1 = u[s];
    T um2 = u[(n - 2) * s], um1 = u[(n - 1) * s], uc = u0, up1 = u1;
    T yp = T(0), acc = T(0);
#pragma unroll 4
    for (int64_t j = 0; j < n; ++j) {
        const int64_t j2 = j + 2;
        const T up2 = j2 < n ? u[j2 * s] : (j2 == n ? u0 : u1);
        const T d = ca * (up1 - um1) + cb * (up2 - um2);
        yp = (d - alpha * yp) * inv[j];
        y[j * s] = yp;
        acc += w[j] * yp;
        um2 = um1;
        um1 = uc;
        uc = up1;
        up1 = up2;
    }
    // Sherman-Morrison scalar: q.y / (1 + q.z) with y_0 = acc, y_{n-1} = y'_{n-1}
    const T sc = kk * (acc + ag * yp);
    // backward: y_j = y'_j - cp_j y_{j+1}; x_j = y_j - sc z_j
    T yn = yp;
    y[(n - 1) * s] = yn - sc * z[n - 1];
#pragma unroll 4
    for (int64_t j = n - 2; j >= 0; --j) {
        yn = y[j * s] - cp[j] * yn;
        y[j * s] = yn - sc * z[j];
    }
    }
}

// Mode 3: the fibers are contiguous rows.  A wave owns 64 rows; tiles of
// 64 rows x RT points (128 bytes per row) go through LDS so that every global
// access is a coalesced 16-byte-per-lane load or store, while each lane still
// walks its own row.  Forward tiles carry a two-point halo (taken modulo n).
// Per-wave LDS: an input tile and an output tile, rows padded by one element.
template <typename T>
struct RowsCfg {
    static constexpr int VE = 16 / int(sizeof(T));    // elements per 16-byte word
    static constexpr int RT = 128 / int(sizeof(T));   // points per tile row
    static constexpr int WPR = RT / VE;               // 16-byte words per tile row
    static constexpr int LD = RT + 3;                 // LDS row stride (tile + halo + pad)
    static constexpr int WAVE_ELEMS = 2 * 64 * LD;
};

template <typename T>
__global__ void __launch_bounds__(256) k_compact_rows(const CompactArgs a, const T *__restrict__ X,
                                                      T *__restrict__ Y, const T *__restrict__ ws) {
    typedef RowsCfg<T> CF;
    constexpr int VE = CF::VE, RT = CF::RT, LD = CF::LD;
    extern __shared__ __align__(16) unsigned char smem_rows[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    T *tin = reinterpret_cast<T *>(smem_rows) + wave * CF::WAVE_ELEMS;
    T *tout = tin + 64 * LD;
    const int64_t n = a.n;
    const int64_t row0 = (int64_t(blockIdx.x) * (blockDim.x >> 6) + wave) * 64;
    if (row0 >= a.nfib) return;                       // whole wave: no LDS shared across waves
    const int64_t nrows = a.nfib - row0 < 64 ? a.nfib - row0 : 64;
    const T *inv = ws, *cp = ws + n, *w = ws + 2 * n, *z = ws + 3 * n;
    const T kk = ws[4 * n], ag = ws[4 * n + 1];
    const T ca = T(a.ca), cb = T(a.cb), alpha = T(a.alpha);
    const int64_t myrow = row0 + (lane < nrows ? lane : nrows - 1);
    const T *urow = X + myrow * n;

    // cooperative tile transfer: lane l moves word l % WPR of rows l / WPR + (64 / WPR) i
    constexpr int WPR = CF::WPR, RPP = 64 / WPR;
    const int wl = lane % WPR, rl = lane / WPR;
    auto load_tile = [&](const T *src, int64_t t0, int cols) {
#pragma unroll
        for (int i = 0; i < WPR; ++i) {
            const int r = rl + RPP * i;
            const int c = wl * VE;
            if (r < nrows && c < cols) {
                const T *g = src + (row0 + r) * n + t0 + c;
                if (c + VE <= cols) {
                    V16 v = ld16(g);
#pragma unroll
                    for (int e = 0; e < VE; ++e) tin[r * LD + c + e] = reinterpret_cast<const T *>(&v)[e];
                } else {
                    for (int e = 0; c + e < cols; ++e) tin[r * LD + c + e] = g[e];
                }
            }
        }
    };
    auto store_tile = [&](T *dst, int64_t t0, int cols) {
#pragma unroll
        for (int i = 0; i < WPR; ++i) {
            const int r = rl + RPP * i;
            const int c = wl * VE;
            if (r < nrows && c < cols) {
                T *g = dst + (row0 + r) * n + t0 + c;
                if (c + VE <= cols) {
                    V16 v;
#pragma unroll
                    for (int e = 0; e < VE; ++e) reinterpret_cast<T *>(&v)[e] = tout[r * LD + c + e];
                    *reinterpret_cast<u32x4 *>(g) = v.u;
                } else {
                    for (int e = 0; c + e < cols; ++e) g[e] = tout[r * LD + c + e];
                }
            }
        }
    };

    // forward sweep over tiles [t0, t0 + cols), halo points t0 + cols, t0 + cols + 1 (mod n)
    T um2 = urow[n - 2], um1 = urow[n - 1], uc = urow[0], up1 = urow[1];
    T yp = T(0), acc = T(0);
    for (int64_t t0 = 0; t0 < n; t0 += RT) {
        const int cols = int(n - t0 < RT ? n - t0 : RT);
        wave_sync();
        load_tile(X, t0, cols);
        // the two halo points of each row (scalar loads, modulo n)
        for (int e = lane; e < 2 * nrows; e += 64) {
            const int r = e >> 1, h = e & 1;
            int64_t c = t0 + cols + h;
            if (c >= n) c -= n;
            tin[r * LD + cols + h] = X[(row0 + r) * n + c];
        }
        wave_sync();
        const T *mine = tin + lane * LD;
        for (int c = 0; c < cols; ++c) {
            const int64_t j = t0 + c;
            const T up2 = mine[c + 2];
            const T d = ca * (up1 - um1) + cb * (up2 - um2);
            yp = (d - alpha * yp) * inv[j];
            tout[lane * LD + c] = yp;
            acc += w[j] * yp;
            um2 = um1;
            um1 = uc;
            uc = up1;
            up1 = up2;
        }
        wave_sync();
        store_tile(Y, t0, cols);
    }
    const T sc = kk * (acc + ag * yp);

    // backward sweep over the same tiles in reverse, in place in Y
    T yn = T(0);
    const int64_t last0 = ((n - 1) / RT) * RT;
    for (int64_t t0 = last0; t0 >= 0; t0 -= RT) {
        const int cols = int(n - t0 < RT ? n - t0 : RT);
        wave_sync();
        load_tile(Y, t0, cols);
        wave_sync();
        const T *mine = tin + lane * LD;
        for (int c = cols - 1; c >= 0; --c) {
            const int64_t j = t0 + c;
            yn = mine[c] - (j == n - 1 ? T(0) : cp[j]) * yn;
            tout[lane * LD + c] = yn - sc * z[j];
        }
        wave_sync();
        store_tile(Y, t0, cols);
    }
}

// The same sweeps for n a multiple of RT (every tile whole): the next tile
// and its halo are loaded into registers while the current one is computed,
// and the RT steps of a tile are unrolled with the tile's coefficients read
// before the recurrence starts.
template <typename T>
__global__ void __launch_bounds__(256) k_compact_rows_full(const CompactArgs a, const T *__restrict__ X,
                                                           T *__restrict__ Y, const T *__restrict__ ws) {
    typedef RowsCfg<T> CF;
    constexpr int VE = CF::VE, RT = CF::RT, LD = CF::LD, WPR = CF::WPR, RPP = 64 / WPR;
    extern __shared__ __align__(16) unsigned char smem_rows[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    T *tin = reinterpret_cast<T *>(smem_rows) + wave * CF::WAVE_ELEMS;
    T *tout = tin + 64 * LD;
    const int64_t n = a.n, ntiles = n / RT;
    const int64_t row0 = (int64_t(blockIdx.x) * (blockDim.x >> 6) + wave) * 64;
    if (row0 >= a.nfib) return;                       // whole wave: no LDS shared across waves
    const int nrows = int(a.nfib - row0 < 64 ? a.nfib - row0 : 64);
    const T *inv = ws, *cp = ws + n, *w = ws + 2 * n, *z = ws + 3 * n;
    const T kk = ws[4 * n], ag = ws[4 * n + 1];
    const T ca = T(a.ca), cb = T(a.cb), alpha = T(a.alpha);
    const int64_t myrow = row0 + (lane < nrows ? lane : nrows - 1);
    const T *urow = X + myrow * n;

    // lane l moves word l % WPR of rows l / WPR + RPP i (rows past the range
    // re-read the last row and are not stored); halo values: lane l holds
    // point t0 + RT + (l & 1) (mod n) of row l / 2 and of row 32 + l / 2
    const int wl = lane % WPR, rl = lane / WPR;
    V16 buf[WPR];
    T halo[2];
    auto rowc = [&](int r) -> int64_t { return row0 + (r < nrows ? r : nrows - 1); };
    auto fetch = [&](const T *src, int64_t t0, bool with_halo) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < WPR; ++i) buf[i] = ld16(src + rowc(rl + RPP * i) * n + t0 + wl * VE);
        if (with_halo) {
            int64_t c = t0 + RT + (lane & 1);
            if (c >= n) c -= n;
#pragma unroll
            for (int h = 0; h < 2; ++h) halo[h] = src[rowc(32 * h + (lane >> 1)) * n + c];
        }
    };
    auto put = [&](bool with_halo) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < WPR; ++i) {
            const int r = rl + RPP * i;
#pragma unroll
            for (int e = 0; e < VE; ++e) tin[r * LD + wl * VE + e] = reinterpret_cast<const T *>(&buf[i])[e];
        }
        if (with_halo) {
#pragma unroll
            for (int h = 0; h < 2; ++h) tin[(32 * h + (lane >> 1)) * LD + RT + (lane & 1)] = halo[h];
        }
    };
    auto store_tile = [&](int64_t t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < WPR; ++i) {
            const int r = rl + RPP * i;
            if (r < nrows) {
                V16 v;
#pragma unroll
                for (int e = 0; e < VE; ++e) reinterpret_cast<T *>(&v)[e] = tout[r * LD + wl * VE + e];
                *reinterpret_cast<u32x4 *>(Y + (row0 + r) * n + t0 + wl * VE) = v.u;
            }
        }
    };

    // forward sweep
    T um2 = urow[n - 2], um1 = urow[n - 1], uc = urow[0], up1 = urow[1];
    T yp = T(0), acc = T(0);
    fetch(X, 0, true);
    for (int64_t t = 0; t < ntiles; ++t) {
        const int64_t t0 = t * RT;
        wave_sync();
        put(true);
        wave_sync();
        T u[RT + 2];
        const T *mine = tin + lane * LD;
#pragma unroll
        for (int c = 0; c < RT + 2; ++c) u[c] = mine[c];
        if (t + 1 < ntiles) fetch(X, t0 + RT, true);
        T ci[RT], cw[RT];
#pragma unroll
        for (int c = 0; c < RT; ++c) {
            ci[c] = inv[t0 + c];
            cw[c] = w[t0 + c];
        }
#pragma unroll
        for (int c = 0; c < RT; ++c) {
            const T up2 = u[c + 2];
            const T d = ca * (up1 - um1) + cb * (up2 - um2);
            yp = (d - alpha * yp) * ci[c];
            tout[lane * LD + c] = yp;
            acc += cw[c] * yp;
            um2 = um1;
            um1 = uc;
            uc = up1;
            up1 = up2;
        }
        wave_sync();
        store_tile(t0);
    }
    const T sc = kk * (acc + ag * yp);

    // backward sweep over the same tiles in reverse, in place in Y (the
    // forward's stores by other lanes of this wave are complete first)
    T yn = T(0);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    fetch(Y, (ntiles - 1) * RT, false);
    for (int64_t t = ntiles - 1; t >= 0; --t) {
        const int64_t t0 = t * RT;
        wave_sync();
        put(false);
        wave_sync();
        T v[RT];
        const T *mine = tin + lane * LD;
#pragma unroll
        for (int c = 0; c < RT; ++c) v[c] = mine[c];
        if (t > 0) fetch(Y, t0 - RT, false);
        T cc[RT], cz[RT];
#pragma unroll
        for (int c = 0; c < RT; ++c) {
            cc[c] = t0 + c == n - 1 ? T(0) : cp[t0 + c];
            cz[c] = z[t0 + c];
        }
#pragma unroll
        for (int c = RT - 1; c >= 0; --c) {
            yn = v[c] - cc[c] * yn;
            tout[lane * LD + c] = yn - sc * cz[c];
        }
        wave_sync();
        store_tile(t0);
    }
}

// ---------------------------------------------------------------------------
// Single-pass sweep.  A_c = tridiag(alpha, 1, alpha) with periodic corners is
// circulant and, for |alpha| < 1/2, factors as
//     A_c = c (I + rho S)(I + rho S^T),  rho = 2 alpha / (1 + sqrt(1 - 4 alpha^2)),
//     c = 1 / (1 + rho^2),  (S y)_j = y_{j+1} (indices mod n),
// so A_c y = d is a cyclic forward recursion f_j = d_j - rho f_{j-1} followed
// by a cyclic backward recursion g_j = f_j - rho g_{j+1}, y = (1 + rho^2) g.
// |rho| < 1 (diagonal dominance, the premise of Sec. 4.2's DistD2): a value
// k steps back (or ahead) enters with weight rho^k, below half the rounding
// unit from k = K on.  A fiber is cut into segments of q or q + 1 points held
// in one thread's registers each.  Every thread runs its recursion from zero;
// the value that enters segment l is then
//     e_{l-1} + m_{l-1} (e_{l-2} + m_{l-2} (e_{l-3} + ...)),
// e the segments' end values and m = (-rho)^length their multipliers, over the
// H segments that hold the last K points, and the thread runs its recursion
// again from it.  Where those are the whole fiber, one turn is enough: further
// ones multiply its sum by 1 / (1 - (-rho)^n).  (Gone round as often as K points
// take, fibers of 5 and 6 points paid for 40 dependent LDS reads: 267 x 5 x 1200
// in double along mode 2 15.5 us, now 8.5; the exact sweeps, prepared, 7.8.)  The
// same backwards.  Each point is read once and written once, whatever n.
// Fibers too long for one block are taken in chunks with K + 2 points more at
// either end, from zero there; the right-hand side is zero at a chunk's two
// outermost points, whose neighbours it does not hold, so that nothing of one
// end reaches the other.
// ---------------------------------------------------------------------------
struct SegArgs {
    int64_t n, stride, nfib, i3, s12, groups;
    int mode, S, q, r, H;        // segments; the first r hold q + 1 points, the others q; segments to look back over
    int K;                       // points a recursion remembers
    int nchunk, M, pad;          // nchunk > 1: chunks of M outputs, S q = M + 2 pad points read for each (r = 0)
    int block;                   // modes 1, 2: 2^block fibers in a block; mode 3: rows in a block
    double ca, cb, rho, scale;   // a / (2h), b / (4h), rho, 1 + rho^2
    double mq, mq1;              // (-rho)^q, (-rho)^(q + 1)
    double turns;                // H == S: 1 / (1 - (-rho)^n), else 1
};

// The two recursions over the thread's points, d -> y, in place: v[0 .. C), or
// v[0 .. C - 1) where the segment is not a long one.  e and eb hold one value
// a thread; segment g of this fiber is at slot (g << shift) + at.  Every
// thread of the block calls it (two barriers).
template <typename T, int C>
__device__ __forceinline__ void seg_solve(const SegArgs &a, T (&v)[C], bool lng, int sg, bool live, T *e, T *eb, int shift,
                                          int at) {
    const T rho = T(a.rho), mq = T(a.mq), mq1 = T(a.mq1), turns = T(a.turns);
    T f = T(0);
#pragma unroll
    for (int i = 0; i < C - 1; ++i) f = v[i] - rho * f;
    f = lng ? v[C - 1] - rho * f : f;
    if (live) e[(sg << shift) + at] = f;
    __syncthreads();
    // forward: what enters from the H segments before
    f = T(0);
    if (live) {
        int g = sg - a.H;
        if (g < 0) g = a.nchunk > 1 ? 0 : g + a.S;
        const int steps = a.nchunk > 1 ? sg - g : a.H;
        for (int m = 0; m < steps; ++m) {
            f = e[(g << shift) + at] + (g < a.r ? mq1 : mq) * f;
            g = g + 1 == a.S ? 0 : g + 1;
        }
        f *= turns;
    }
#pragma unroll
    for (int i = 0; i < C; ++i) {
        f = v[i] - rho * f;
        v[i] = f;
    }
    f = lng ? v[C - 1] : T(0);
#pragma unroll
    for (int i = C - 2; i >= 0; --i) f = v[i] - rho * f;
    if (live) eb[(sg << shift) + at] = f;
    __syncthreads();
    f = T(0);
    if (live) {
        int g = sg + a.H;
        if (g >= a.S) g = a.nchunk > 1 ? a.S - 1 : g - a.S;
        const int steps = a.nchunk > 1 ? g - sg : a.H;
        for (int m = 0; m < steps; ++m) {
            f = eb[(g << shift) + at] + (g < a.r ? mq1 : mq) * f;
            g = g == 0 ? a.S - 1 : g - 1;
        }
        f *= turns;
    }
    const T scale = T(a.scale);
    if (lng) {
        f = v[C - 1] - rho * f;
        v[C - 1] = scale * f;
    }
#pragma unroll
    for (int i = C - 2; i >= 0; --i) {
        f = v[i] - rho * f;
        v[i] = scale * f;
    }
}

// Modes 1 and 2: a block takes F = 2^a.block neighbouring fibers (so F values in a
// row are read at every point), thread (segment, fiber) the segment's points.
// The two points on either side of a segment come through LDS from the threads
// that hold them.  Bound by memory: all of a block's reads are in flight at
// once, and its arithmetic hides behind other blocks' (2 to 4 on a compute
// unit).  Blocks of neighbouring fibers run on one XCD: where rows start
// inside a cache line, the two halves of a line meet in one L2 (181 x 250 x
// 300 float32: 21 us a mode against 27 to 31 in launch order; 400 x 333 x 511
// float64 0.26 / 0.23 ms against 0.34 / 0.31).  F of 16 (128 or 64 bytes) and
// segments of 16 points measured best of F 16 to 64 and 8 or 16 points:
// mode 2 of 512^3 float64 0.387 ms (5.5 TB/s, the rate of a plain copy);
// one lane a fiber, walked from end to end, took 0.43 ms there, and the exact
// sweeps, which odd lengths took before, 0.12 to 0.19 ms at 181 x 250 x 300.
template <typename T, int C>
__global__ void __launch_bounds__(1024) k_compact_lines(const SegArgs a, const T *__restrict__ X, T *__restrict__ Y) {
    extern __shared__ __align__(16) unsigned char smem_seg[];
    const int F = 1 << a.block, nt = a.S << a.block;
    T *first0 = reinterpret_cast<T *>(smem_seg), *first1 = first0 + nt, *last0 = first1 + nt, *last1 = last0 + nt;
    T *e = last1 + nt, *eb = e + nt;
    const int me = int(threadIdx.x), fi = me & (F - 1), sg = me >> a.block;
    const bool lng = sg < a.r || a.q == C;               // C points, else C - 1
    const int before = (((sg == 0 ? a.S : sg) - 1) << a.block) + fi;
    const int after = ((sg + 1 >= a.S ? 0 : sg + 1) << a.block) + fi;
    const T ca = T(a.ca), cb = T(a.cb);
    const int64_t s = a.stride;
    for (int64_t g0 = blockIdx.x; g0 < a.groups; g0 += gridDim.x) {
        int64_t grp = g0;
        if (g0 < (a.groups & ~int64_t(7))) grp = (g0 & 7) * (a.groups >> 3) + (g0 >> 3);
        const int64_t chunk = a.nchunk > 1 ? grp % a.nchunk : 0;
        const int64_t f = ((a.nchunk > 1 ? grp / a.nchunk : grp) << a.block) + fi;
        const bool live = sg < a.S && f < a.nfib;
        int64_t base = f;
        if (a.mode == 2) {
            if (a.nfib < (int64_t(1) << 31)) {
                const uint32_t line = uint32_t(f) / uint32_t(a.i3);
                base = int64_t(line) * a.s12 + (uint32_t(f) - line * uint32_t(a.i3));
            } else {
                base = (f / a.i3) * a.s12 + f % a.i3;
            }
        }
        // first point of the segment; in chunks modulo n (M + 2 pad points may go round)
        const int64_t j0 = chunk * a.M - (a.nchunk > 1 ? a.pad : 0) + int64_t(sg) * a.q + (sg < a.r ? sg : a.r);
        T u[C + 4];
        if (live) {
            if (a.nchunk == 1) {
                const T *p = X + base + j0 * s;
#pragma unroll
                for (int i = 0; i < C - 1; ++i) u[i + 2] = p[i * s];
                u[C + 1] = lng ? p[(C - 1) * s] : T(0);
            } else {
                int64_t j = j0 % a.n;
                if (j < 0) j += a.n;
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    u[i + 2] = X[base + j * s];
                    j = j + 1 == a.n ? 0 : j + 1;
                }
            }
            first0[me] = u[2];
            first1[me] = u[3];
            last0[me] = lng ? u[C] : u[C - 1];
            last1[me] = lng ? u[C + 1] : u[C];
        }
        __syncthreads();
        T v[C];
        if (live) {
            u[0] = last0[before];
            u[1] = last1[before];
            const T n0 = first0[after], n1 = first1[after];
            u[C + 1] = lng ? u[C + 1] : n0;
            u[C + 2] = lng ? n0 : n1;
            u[C + 3] = n1;
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = ca * (u[i + 3] - u[i + 1]) + cb * (u[i + 4] - u[i]);
            if (a.nchunk > 1 && sg == 0) v[0] = v[1] = T(0);
            if (a.nchunk > 1 && sg == a.S - 1) v[C - 1] = v[C - 2] = T(0);
        } else {
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = T(0);
        }
        seg_solve<T, C>(a, v, lng, sg, live, e, eb, a.block, fi);
        if (live) {
            if (a.nchunk == 1) {
                T *p = Y + base + j0 * s;
#pragma unroll
                for (int i = 0; i < C - 1; ++i) p[i * s] = v[i];
                if (lng) p[(C - 1) * s] = v[C - 1];
            } else {
                const int64_t lo = chunk * a.M, hi = lo + a.M < a.n ? lo + a.M : a.n;
#pragma unroll
                for (int i = 0; i < C; ++i)
                    if (j0 + i >= lo && j0 + i < hi) Y[base + (j0 + i) * s] = v[i];
            }
        }
        __syncthreads();
    }
}

// Mode 3: the fibers are contiguous rows.  A block takes R = a.block neighbouring
// rows, brings them into LDS as one contiguous run (16 bytes a lane where the
// runs are aligned: VEC), threads (row, segment) take their points and the two
// on either side from there and put the result back, and the run leaves as it
// came.  Positions are padded by one element every 8, so that the segments of
// neighbouring lanes start in different banks.  Bound by memory: 512^3 float64
// 0.383 ms (5.6 TB/s; one wave a row with a warm-up of K points in every lane
// 0.39 to 0.44 ms, for power-of-two rows alone), 181 x 250 x 300 float32
// 26 us (exact sweeps 122 us).  256 threads a block; 64 to 1024 measured
// within 3 % or worse.
template <typename T, int C, bool VEC>
__global__ void __launch_bounds__(1024) k_compact_rows1p(const SegArgs a, const T *__restrict__ X, T *__restrict__ Y) {
    constexpr int VE = 16 / int(sizeof(T));
    extern __shared__ __align__(16) unsigned char smem_seg[];
    const int R = a.block, width = a.nchunk > 1 ? a.S * a.q : int(a.n), run = R * width;
    auto pos = [](int j) __attribute__((always_inline)) { return j + (j >> 3); };
    T *ub = reinterpret_cast<T *>(smem_seg);
    T *e = ub + pos(run) + 1, *eb = e + R * a.S;
    const int nt = int(blockDim.x), tid = int(threadIdx.x);
    const int row = tid / a.S, sg = tid - row * a.S;
    const bool lng = sg < a.r || a.q == C;               // C points, else C - 1
    const int j0 = sg * a.q + (sg < a.r ? sg : a.r), rb = row * width;
    const int jn = j0 + (lng ? C : C - 1);               // the point after the segment
    const T ca = T(a.ca), cb = T(a.cb);
    for (int64_t grp = blockIdx.x; grp < a.groups; grp += gridDim.x) {
        const int64_t chunk = a.nchunk > 1 ? grp % a.nchunk : 0;
        const int64_t r0 = (a.nchunk > 1 ? grp / a.nchunk : grp) * R;
        const int rows = int(a.nfib - r0 < R ? a.nfib - r0 : R);
        const T *src = X + r0 * a.n;
        T *dst = Y + r0 * a.n;
        const int have = rows * width;
        if (a.nchunk > 1) {
            const int64_t c0 = chunk * a.M - a.pad;
            for (int k = tid; k < width; k += nt) {
                int64_t j = (c0 + k) % a.n;
                if (j < 0) j += a.n;
                ub[pos(k)] = src[j];
            }
        } else if (VEC) {
            for (int k = tid * VE; k < have; k += nt * VE) {
                if (k + VE <= have) {
                    V16 w;
                    w.u = *reinterpret_cast<const u32x4 *>(src + k);
#pragma unroll
                    for (int i = 0; i < VE; ++i) ub[pos(k + i)] = reinterpret_cast<const T *>(&w)[i];
                } else {
                    for (int i = 0; k + i < have; ++i) ub[pos(k + i)] = src[k + i];
                }
            }
        } else {
            for (int k = tid; k < have; k += nt) ub[pos(k)] = src[k];
        }
        __syncthreads();
        const bool live = row < rows;
        T v[C];
        if (live) {
            T u[C + 4];
            auto at = [&](int j) __attribute__((always_inline)) {   // j in [-2, width + 1]
                return ub[pos(rb + (j < 0 ? j + width : j >= width ? j - width : j))];
            };
            u[0] = at(j0 - 2);
            u[1] = at(j0 - 1);
#pragma unroll
            for (int i = 0; i < C - 1; ++i) u[i + 2] = ub[pos(rb + j0 + i)];
            const T n0 = at(jn), n1 = at(jn + 1);
            u[C + 1] = lng ? ub[pos(rb + j0 + C - 1)] : n0;
            u[C + 2] = lng ? n0 : n1;
            u[C + 3] = n1;
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = ca * (u[i + 3] - u[i + 1]) + cb * (u[i + 4] - u[i]);
            if (a.nchunk > 1 && sg == 0) v[0] = v[1] = T(0);
            if (a.nchunk > 1 && sg == a.S - 1) v[C - 1] = v[C - 2] = T(0);
        } else {
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = T(0);
        }
        seg_solve<T, C>(a, v, lng, sg, live, e, eb, 0, row * a.S);
        // every thread has read its points (two barriers ago): y takes their place
        if (live) {
#pragma unroll
            for (int i = 0; i < C - 1; ++i) ub[pos(rb + j0 + i)] = v[i];
            if (lng) ub[pos(rb + j0 + C - 1)] = v[C - 1];
        }
        __syncthreads();
        if (a.nchunk > 1) {
            const int64_t lo = chunk * a.M, hi = lo + a.M < a.n ? lo + a.M : a.n;
            for (int k = tid; k < int(hi - lo); k += nt) dst[lo + k] = ub[pos(k + a.pad)];
        } else if (VEC) {
            for (int k = tid * VE; k < have; k += nt * VE) {
                if (k + VE <= have) {
                    V16 w;
#pragma unroll
                    for (int i = 0; i < VE; ++i) reinterpret_cast<T *>(&w)[i] = ub[pos(k + i)];
                    *reinterpret_cast<u32x4 *>(dst + k) = w.u;
                } else {
                    for (int i = 0; k + i < have; ++i) dst[k + i] = ub[pos(k + i)];
                }
            }
        } else {
            for (int k = tid; k < have; k += nt) dst[k] = ub[pos(k)];
        }
        __syncthreads();
    }
}

// Modes 1 and 2 with points far apart (512 KiB and more) and many of them: one
// lane per fiber walks it from end to end, so that the whole chip reads one
// plane of the field after the other, where the segments of k_compact_lines
// would keep every plane open at once (512^3 float64, 2 MiB apart: 0.437 ms
// against 0.492; 1024 x 256 x 256 0.201 against 0.254; with 400 points or
// fewer, or 4 KiB apart, the segments win: 0.26 against 0.27, 0.39 against 0.43).
// The forward recursion runs K + L points ahead of the outputs in a register
// window F[K + L]; every L points the backward recursion runs over the window
// from its far end and the first L values are stored.  The stencil reads of a
// block are issued before its recursion.  The warm-up reads the K + 4 points
// before point 0 (cyclically); the window past the fiber's end reuses
// f_0 .. f_{K-1} kept in registers, so a fiber is read n + K + 8 times.
template <typename T, int K, int L>
__global__ void __launch_bounds__(256) k_compact_march(const SegArgs a, const T *__restrict__ X,
                                                       T *__restrict__ Y) {
    const int64_t n = a.n, s = a.stride;
    const T ca = T(a.ca), cb = T(a.cb), rho = T(a.rho), scale = T(a.scale);
    for (int64_t f = int64_t(blockIdx.x) * 256 + threadIdx.x; f < a.nfib; f += int64_t(gridDim.x) * 256) {
        const int64_t base = a.mode == 1 ? f : (f / a.i3) * a.s12 + f % a.i3;
        const T *u = X + base;
        T *y = Y + base;
        // the stencil stream: point j needs u_{j-2} .. u_{j+2} (mod n); jn is
        // the index (mod n) of the next value to read
        int64_t jn = n - K + 2;
        T um2 = u[(n - K - 2) * s], um1 = u[(n - K - 1) * s], uc = u[(n - K) * s], up1 = u[(n - K + 1) * s];
        auto next_index = [&]() __attribute__((always_inline)) {
            const int64_t j = jn;
            jn = jn + 1 == n ? 0 : jn + 1;
            return j;
        };
        auto step = [&](T up2) __attribute__((always_inline)) {
            const T d = ca * (up1 - um1) + cb * (up2 - um2);
            um2 = um1;
            um1 = uc;
            uc = up1;
            up1 = up2;
            return d;
        };
        // the backward recursion over the window from its far end; the first
        // L values are the outputs of points b .. b + L - 1; then the window
        // moves on by L
        auto emit = [&](T (&W)[K + L], int64_t b0) __attribute__((always_inline)) {
            T g = T(0);
#pragma unroll
            for (int i = K + L - 1; i >= L; --i) g = W[i] - rho * g;
            T out[L];
#pragma unroll
            for (int i = L - 1; i >= 0; --i) {
                g = W[i] - rho * g;
                out[i] = scale * g;
            }
#pragma unroll
            for (int i = 0; i < L; ++i)
                if (b0 + i < n) y[(b0 + i) * s] = out[i];
#pragma unroll
            for (int i = 0; i < K; ++i) W[i] = W[i + L];
        };
        // forward warm-up over the K points before point 0
        T fprev = T(0);
#pragma unroll 8
        for (int t = 0; t < K; ++t) fprev = step(u[next_index() * s]) - rho * fprev;
        // F[i] = f_{b + i}: first f_0 .. f_{K-1}, kept (fs) for the window
        // past the fiber's end (f is cyclic: f_{n + i} = f_i), so the last
        // blocks read nothing again
        T F[K + L], fs[K];
#pragma unroll
        for (int t = 0; t < K; ++t) {
            fprev = step(u[next_index() * s]) - rho * fprev;
            F[t] = fprev;
            fs[t] = fprev;
        }
        // n and K are multiples of L (host): the last K / L blocks take the
        // whole new part of their window from fs
        static_assert(K % L == 0, "window blocks");
        int64_t b = 0;
        for (; b + K + L <= n; b += L) {
            T v[L];
#pragma unroll
            for (int t = 0; t < L; ++t) v[t] = u[next_index() * s];
#pragma unroll
            for (int t = 0; t < L; ++t) {
                fprev = step(v[t]) - rho * fprev;
                F[K + t] = fprev;
            }
            emit(F, b);
        }
#pragma unroll
        for (int m = 0; m < K / L; ++m, b += L) {
#pragma unroll
            for (int t = 0; t < L; ++t) F[K + t] = fs[m * L + t];
            emit(F, b);
        }
    }
}

// Points after which a recursion has forgotten its start (rho^K below half the
// rounding unit), 0 where that takes more than SEG_KMAX: the exact sweeps run.
// alpha = 1/3 takes 39 points in float64 and 19 in float32.
constexpr int SEG_KMAX = 64;
inline int seg_memory(double rho, int dtype) {
    const double r = fabs(rho), most = dtype == TTM_F64 ? 0x1p-54 : 0x1p-25;
    double w = r;
    for (int k = 1; k <= SEG_KMAX; ++k, w *= r)
        if (w <= most) return k;
    return 0;
}

template <typename T>
int single_pass(const SegArgs &in, const T *X, T *Y, hipStream_t st) {
    SegArgs a = in;
    // KT: the window of k_compact_march, which needs whole blocks of 8 points and 2 KT of them
    constexpr int VE = 16 / int(sizeof(T)), KT = sizeof(T) == 8 ? 40 : 24;
    if (a.mode != 3 && a.n > 448 && a.n % 8 == 0 && a.K <= KT && a.stride * int64_t(sizeof(T)) >= (512 << 10) && a.nfib >= 65536)
        return launch("ttm_compact", st, [&] {
            hipLaunchKernelGGL((k_compact_march<T, KT, 8>), dim3(unsigned(ceil_div(a.nfib, 256))), dim3(256), 0, st, a, X, Y);
        });
    int flog = a.mode == 3 ? 0 : 4;
    const int most = 1024 >> flog;   // segments in a block
    // the longest segments (16, 8, 4 points; 8, 4 for rows) that the fiber
    // can be cut into with no other length than C and C - 1; n = 5 alone has
    // none and takes 3 + 2
    int C = a.mode == 3 ? 8 : 16;
    while (C > 4 && a.n / ceil_div(a.n, C) < C - 1) C >>= 1;
    if (a.n == 5) C = 3;
    int64_t S = ceil_div(a.n, C);
    a.nchunk = 1;
    if (S > most) {
        S = most;
        a.pad = a.K + 2;
        a.M = int(S) * C - 2 * a.pad;
        a.nchunk = int(ceil_div(a.n, a.M));
        a.q = C;
    } else {
        a.q = int(a.n / S);
        a.r = int(a.n % S);
    }
    a.S = int(S);
    a.H = int(ceil_div(a.K, a.q));
    a.turns = 1.0;
    if (a.nchunk == 1 && a.H >= a.S) {
        a.H = a.S;
        a.turns = 1.0 / (1.0 - pow(-a.rho, double(a.n)));
    }
    a.mq = pow(-a.rho, double(a.q));
    a.mq1 = pow(-a.rho, double(a.q + 1));
    size_t lds;
    int nt;
    bool vec = false;
    if (a.mode == 3) {
        int R = 1;
        if (a.nchunk == 1) {
            // about 256 threads, fewer where that would leave compute units without a block
            R = std::max(1, 256 / a.S);
            while (R > VE && a.nfib < int64_t(R) * 1024) R >>= 1;
            if (R >= VE) R -= R % VE;
        }
        vec = a.nchunk == 1 && (R * a.n) % VE == 0 && aligned(X, 16) && aligned(Y, 16);
        a.block = R;
        const int run = R * (a.nchunk > 1 ? a.S * a.q : int(a.n));
        lds = (size_t(run + (run >> 3) + 1) + 2 * size_t(R) * a.S) * sizeof(T);
        nt = int(round_up(R * a.S, 64));
        a.groups = ceil_div(a.nfib, R) * a.nchunk;
    } else {
        // up to 512 threads, fewer where that would leave compute units without a block
        while ((a.S << (flog + 1)) <= 512 && (a.nfib >> (flog + 1)) >= 1024) ++flog;
        a.block = flog;
        lds = 6 * (size_t(a.S) << flog) * sizeof(T);
        nt = int(round_up(int64_t(a.S) << flog, 64));
        a.groups = ceil_div(a.nfib, int64_t(1) << flog) * a.nchunk;
    }
    const unsigned blocks = unsigned(std::min<int64_t>(a.groups, 1 << 20));
    void (*kern)(const SegArgs, const T *, T *);
    auto pick = [&](auto c) {
        constexpr int CC = decltype(c)::value;
        if (a.mode == 3) return vec ? k_compact_rows1p<T, CC, true> : k_compact_rows1p<T, CC, false>;
        return k_compact_lines<T, CC>;
    };
    switch (C) {
        case 3: kern = pick(std::integral_constant<int, 3>()); break;
        case 4: kern = pick(std::integral_constant<int, 4>()); break;
        case 8: kern = pick(std::integral_constant<int, 8>()); break;
        default: kern = k_compact_lines<T, 16>; break;
    }
    if (lds > (48 << 10) && hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                int(lds)) != hipSuccess)
        return TTM_ERR_HIP;
    return launch("ttm_compact", st, [&] { hipLaunchKernelGGL(kern, dim3(blocks), dim3(nt), lds, st, a, X, Y); });
}

}  // namespace

}  // namespace ttm

using namespace ttm;

extern "C" {

size_t ttm_compact_workspace_size(int64_t n, int dtype) {
    const size_t es = dtype_size(dtype);
    if (n < 3 || (dtype != TTM_F64 && dtype != TTM_F32)) return 0;
    return (size_t(4 * n + 2) * es + 255) & ~size_t(255);
}

int ttm_compact_apply(const int64_t *dims, int mode, const void *X, void *Y, int dtype, const ttm_compact_coef *coef,
                      void *ws, size_t ws_bytes, int prepared, void *stream) {
    if (!dims || !X || !Y || !coef) return TTM_ERR_INVALID_ARG;
    if (mode < 1 || mode > 3) return TTM_ERR_INVALID_ARG;
    if (dtype != TTM_F64 && dtype != TTM_F32) return TTM_ERR_UNSUPPORTED;
    int64_t total = 1;
    for (int k = 0; k < 3; ++k) {
        if (dims[k] < 1) return TTM_ERR_INVALID_ARG;
        total = checked_prod(total, dims[k]);
        if (total < 0) return TTM_ERR_INVALID_ARG;
    }
    const int64_t n = dims[mode - 1];
    if (n < 3) return TTM_ERR_UNSUPPORTED;
    if (!(coef->h != 0.0) || !isfinite(coef->h) || !isfinite(coef->alpha) || !isfinite(coef->a) ||
        !isfinite(coef->b) || !(fabs(coef->alpha) < 0.5))
        return TTM_ERR_INVALID_ARG;
    const size_t es = dtype_size(dtype);
    if (!aligned(X, es) || !aligned(Y, es)) return TTM_ERR_INVALID_ARG;
    if (overlaps(X, size_t(total) * es, Y, size_t(total) * es)) return TTM_ERR_ALIAS;
    const size_t need = ttm_compact_workspace_size(n, dtype);
    if (!ws || ws_bytes < need || !aligned(ws, 16)) return TTM_ERR_WORKSPACE;
    if (overlaps(ws, need, Y, size_t(total) * es) || overlaps(ws, need, X, size_t(total) * es))
        return TTM_ERR_ALIAS;

    CompactArgs a;
    a.n = n;
    a.mode = mode;
    a.stride = mode == 1 ? dims[1] * dims[2] : (mode == 2 ? dims[2] : 1);
    a.nfib = total / n;
    a.i3 = dims[2];
    a.s12 = dims[1] * dims[2];
    a.ca = coef->a / (2.0 * coef->h);
    a.cb = coef->b / (4.0 * coef->h);
    a.alpha = coef->alpha;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // The single pass wherever the recursions forget their start soon enough:
    // a rule on alpha and the type alone, so that a prepared call, whose
    // workspace an earlier call with the same fiber length, coef and dtype
    // left, takes the same path as that call, and nothing has to be prepared
    // for the single pass.
    const double alpha = coef->alpha;
    // (the other form of the root, (1 - sqrt(1 - 4 alpha^2)) / (2 alpha), loses
    // its digits to cancellation where alpha is small)
    const double rho = 2.0 * alpha / (1.0 + sqrt(1.0 - 4.0 * alpha * alpha));
    if (const int K = seg_memory(rho, dtype)) {
        SegArgs sa{};
        sa.n = n;
        sa.stride = a.stride;
        sa.nfib = a.nfib;
        sa.i3 = a.i3;
        sa.s12 = a.s12;
        sa.mode = mode;
        sa.K = K;
        sa.ca = a.ca;
        sa.cb = a.cb;
        sa.rho = rho;
        sa.scale = 1.0 + rho * rho;
        return dtype == TTM_F64 ? single_pass(sa, static_cast<const double *>(X), static_cast<double *>(Y), st)
                                : single_pass(sa, static_cast<const float *>(X), static_cast<float *>(Y), st);
    }
    const unsigned blocks = unsigned(ceil_div(a.nfib, 256));
    // mode 3: 4 waves of 64 rows per block, each wave with its own LDS tiles
    const unsigned row_blocks = unsigned(ceil_div(a.nfib, 256));
    const size_t prep_lds = n <= COMPACT_PREP_LDS_MAX ? size_t(16 * n) : 0;
    {
        static std::atomic<uint64_t> prep_attr[2];
        const int k = dtype == TTM_F64 ? 0 : 1;
        const void *fn = dtype == TTM_F64 ? reinterpret_cast<const void *>(&k_compact_prep<double>)
                                          : reinterpret_cast<const void *>(&k_compact_prep<float>);
        if (int rc = ensure_lds_limit(fn, size_t(16 * COMPACT_PREP_LDS_MAX), prep_attr[k])) return rc;
    }
    // mode 3: whole tiles take the prefetching kernel
    const bool full_tiles = n % (dtype == TTM_F64 ? RowsCfg<double>::RT : RowsCfg<float>::RT) == 0;
    if (mode == 3) {
        static std::atomic<uint64_t> attr_set[2][2];
        const int k = dtype == TTM_F64 ? 0 : 1, f = full_tiles ? 1 : 0;
        const void *fn = dtype == TTM_F64
                             ? (full_tiles ? reinterpret_cast<const void *>(&k_compact_rows_full<double>)
                                           : reinterpret_cast<const void *>(&k_compact_rows<double>))
                             : (full_tiles ? reinterpret_cast<const void *>(&k_compact_rows_full<float>)
                                           : reinterpret_cast<const void *>(&k_compact_rows<float>));
        const size_t bytes = dtype == TTM_F64 ? 4 * RowsCfg<double>::WAVE_ELEMS * sizeof(double)
                                              : 4 * RowsCfg<float>::WAVE_ELEMS * sizeof(float);
        if (int rc = ensure_lds_limit(fn, bytes, attr_set[k][f])) return rc;
    }
    int rc = TTM_OK;
    if (dtype == TTM_F64) {
        if (!prepared)
            rc = launch("ttm_compact_prep", st, [&] {
                hipLaunchKernelGGL(k_compact_prep<double>, dim3(1), dim3(64), prep_lds, st, n, coef->alpha,
                                   static_cast<double *>(ws));
            });
        if (rc == TTM_OK && mode == 3)
            rc = launch("ttm_compact", st, [&] {
                hipLaunchKernelGGL(full_tiles ? k_compact_rows_full<double> : k_compact_rows<double>, dim3(row_blocks), dim3(256),
                                   4 * RowsCfg<double>::WAVE_ELEMS * sizeof(double), st, a,
                                   static_cast<const double *>(X), static_cast<double *>(Y),
                                   static_cast<const double *>(ws));
            });
        else if (rc == TTM_OK)
            rc = launch("ttm_compact", st, [&] {
                hipLaunchKernelGGL(k_compact<double>, dim3(blocks), dim3(256), 0, st, a, static_cast<const double *>(X),
                                   static_cast<double *>(Y), static_cast<const double *>(ws));
            });
    } else {
        if (!prepared)
            rc = launch("ttm_compact_prep", st, [&] {
                hipLaunchKernelGGL(k_compact_prep<float>, dim3(1), dim3(64), prep_lds, st, n, coef->alpha,
                                   static_cast<float *>(ws));
            });
        if (rc == TTM_OK && mode == 3)
            rc = launch("ttm_compact", st, [&] {
                hipLaunchKernelGGL(full_tiles ? k_compact_rows_full<float> : k_compact_rows<float>, dim3(row_blocks), dim3(256),
                                   4 * RowsCfg<float>::WAVE_ELEMS * sizeof(float), st, a,
                                   static_cast<const float *>(X), static_cast<float *>(Y),
                                   static_cast<const float *>(ws));
            });
        else if (rc == TTM_OK)
            rc = launch("ttm_compact", st, [&] {
                hipLaunchKernelGGL(k_compact<float>, dim3(blocks), dim3(256), 0, st, a, static_cast<const float *>(X),
                                   static_cast<float *>(Y), static_cast<const float *>(ws));
            });
    }
    return rc;
}

}  // extern "C"
