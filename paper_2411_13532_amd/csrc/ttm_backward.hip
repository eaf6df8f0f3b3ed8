// ttm_backward.hip -- adjoint of the chain Y = X x1 A x2 B x3 C.
//
// Given G = dL/dY (J1 x J2 x J3), every gradient is a contraction of G
// with the inputs, evaluated as a short sequence of unfolded products on
// the matrix cores (k_gemm), each reading its operands in place:
//   W  = X x3 C                 (I1 I2 x J3)      = X_(12) C^T
//   V  = W x2 B = X x2 B x3 C   (I1 x J2 x J3)    per i1: B W[i1]
//   H  = G x1 A^T               (I1 x J2 x J3)    = A^T G_(1)
//   R  = H x2 B^T               (I1 x I2 x J3)    per i1: B^T H[i1]
//   dX = R x3 C^T               (I1 x I2 x I3)    = R_(12) C
//   dA = G_(1) V_(1)^T          (J1 x I1)
//   dB = sum_{i1,j3} H[i1,j2,j3] W[i1,i2,j3]       (J2 x I2)
//   dC = R_(3) X_(3)^T          (J3 x I3)
// so dX = G x1 A^T x2 B^T x3 C^T and each factor gradient contracts G with
// the input chain that skips that factor.  Long contractions (over I1*I2 or
// I1*J3) are split over workgroups and summed in a fixed order.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "ttm_gemm.hpp"
#include "ttm_host.hpp"

namespace ttm {

namespace {

struct BwdPlan {
    int math;
    size_t esz;
    int64_t I1, I2, I3, J1, J2, J3, NN;
    bool need_w, need_v, need_h, need_r;
    size_t off_W, off_V, off_H, off_R, off_P[3], total;   // P: the splits of dA, dB, dC
    // the streaming kernels: J3 <= 64 for W, dX and dC (the X-sized products),
    // J2 <= 64 too for V and R, rows of at least one 16-byte group
    bool stream, stream_vr;
    int dc_splits;
    int64_t dc_rows;
    // float32 with J <= 32, I3 in {256, 512} and I2 a multiple of 4:
    // the three fused kernels (ncg = I3 / 64), with their own workspace layout
    bool fused;
    int ncg;
    size_t f_off_B, f_off_C, f_total;
};

constexpr int64_t KT_F32 = 32, KT_F64 = 16;
constexpr int SK_WAVES = 4;   // waves of a streaming kernel's workgroup (but dC's)

struct SplitK {
    int ks;
    int64_t per;
};

SplitK choose_split(int64_t M, int64_t N, int64_t K, int64_t batch, int64_t KT) {
    const int64_t tiles = ceil_div(M, 64) * ceil_div(N, 64) * batch;
    int64_t ks = ceil_div(512, tiles);
    ks = std::max<int64_t>(1, std::min<int64_t>(ks, ceil_div(K, KT * 4)));
    ks = std::min<int64_t>(ks, 256);
    const int64_t per = round_up(ceil_div(K, ks), KT);
    return {int(ceil_div(K, per)), per};
}

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

void make_bwd_plan(const ttm_shape &s, int math, bool dX, bool dA, bool dB, bool dC, BwdPlan &p) {
    p = BwdPlan();
    p.math = math;
    p.esz = math == TTM_MATH_F64 ? 8 : 4;
    p.I1 = s.I[0]; p.I2 = s.I[1]; p.I3 = s.I[2];
    p.J1 = s.J[0]; p.J2 = s.J[1]; p.J3 = s.J[2];
    p.NN = p.J2 * p.J3;
    p.need_w = dA || dB;
    p.need_v = dA;
    p.need_h = dX || dB || dC;
    p.need_r = dX || dC;
    const int64_t KT = math == TTM_MATH_F64 ? KT_F64 : KT_F32, VE = int64_t(16 / p.esz);
    const int64_t M = p.I1 * p.I2;
    // (the column tiles of dX and dC, and R's row tiles, are grid y: at most
    // 65535 of them; the general product has its tiles along grid x)
    constexpr int64_t YMAX = 65535;
    p.stream = p.J3 <= 64 && p.J3 >= VE && p.I3 >= VE && M < (int64_t(1) << 31) && ceil_div(p.I3, 64 * VE) <= YMAX;
    p.stream_vr = p.J3 <= 64 && p.J2 <= 64 && p.I2 >= VE && ceil_div(p.I2, 32 * SK_WAVES) <= YMAX && p.I1 < (int64_t(1) << 31);
    // partials of the split contractions
    int64_t part[3] = {0, 0, 0};
    if (dA) {
        SplitK k = choose_split(p.J1, p.I1, p.NN, 1, KT);
        if (k.ks > 1) part[0] = k.ks * p.J1 * p.I1;
    }
    if (dB) {
        SplitK k = choose_split(p.J2, p.I2, p.I1 * p.J3, 1, KT);
        if (k.ks > 1) part[1] = k.ks * p.J2 * p.I2;
    }
    if (dC && p.stream) {
        // one workgroup per compute unit and column tile, a split of at least
        // 64 rows (32 per half)
        const int64_t s0 = std::max<int64_t>(1, std::min<int64_t>(ceil_div(256, ceil_div(p.I3, 64 * VE)), ceil_div(M, 64)));
        p.dc_rows = round_up(ceil_div(M, s0), 8);
        p.dc_splits = int(ceil_div(M, p.dc_rows));
        if (p.dc_splits > 1) part[2] = p.dc_splits * p.J3 * p.I3;
    } else if (dC) {
        SplitK k = choose_split(p.J3, p.I3, p.I1 * p.I2, 1, KT);
        if (k.ks > 1) part[2] = k.ks * p.J3 * p.I3;
    }
    size_t off = 0;
    auto take = [&](bool need, int64_t elems) -> size_t {
        if (!need) return 0;
        size_t o = off;
        off = al256(off + size_t(elems) * p.esz);
        return o;
    };
    p.off_W = take(p.need_w, p.I1 * p.I2 * p.J3);
    p.off_V = take(p.need_v, p.I1 * p.NN);
    p.off_H = take(p.need_h, p.I1 * p.NN);
    p.off_R = take(p.need_r, p.I1 * p.I2 * p.J3);
    for (int i = 0; i < 3; ++i) p.off_P[i] = take(part[i] > 0, part[i]);
    p.total = off;

    p.fused = math == TTM_MATH_F32 && p.J1 <= 32 && p.J2 <= 32 && p.J3 <= 32 &&
              (p.I3 == 256 || p.I3 == 512) && p.I2 % 4 == 0 && p.I2 < (int64_t(1) << 24) &&
              p.I1 < (int64_t(1) << 31);
    p.ncg = int(p.I3 / 64);
    off = 0;
    p.f_off_B = take(p.fused, p.I1 * p.J2 * p.I2);
    p.f_off_C = take(p.fused, p.I1 * p.J3 * p.I3);
    p.f_total = off;
}

GemmArgs gargs() {
    GemmArgs a;
    memset(&a, 0, sizeof a);
    a.P = 1;
    return a;
}

// ---------------------------------------------------------------------------
// Streaming kernels for the products of the adjoint with J3 (for V and R also
// J2) at most 64, in float and double, for any row length and alignment of at
// least one 16-byte group.  Rows r = (i1, i2) of X, dX (I3 long) and of W, R
// (J3 long).  Each lane reads 16 bytes (VE values) of a row straight into a
// 16 x 16 x 4 matrix-core operand: which k (or n) value a (lane group,
// element) slot carries is free as long as both operands agree, so one access
// feeds VE products.  A group that would end past its row starts VE before the
// row's end instead: where its values are k slots those before its place are
// zeroed, where they are output columns a neighbour's are formed twice, to the
// same bits.  No LDS in the loops, no barriers: the small operands (C, R, B,
// H) come through the caches, and enough waves are resident to cover the trips
// of the X-sized one, whose bytes bound the three kernels that touch it.
// 200 x 190 x 230 -> 40 x 48 x 36 in float, the general GEMM's time first:
// W 47.8, now 25.9 us; dX 35.0, now 17.5; dC 33.6, now 16.6; V 16.0, now 9.9;
// R 12.7, now 8.7.
// ---------------------------------------------------------------------------
template <typename T> struct Sk;
template <> struct Sk<float> {
    typedef f32x4 acc;
    static constexpr int VE = 4;
    __device__ static float at(const V16 &v, int e) { return v.f[e]; }
    __device__ static void zero(V16 &v, int e) { v.f[e] = 0.f; }
    __device__ static f32x4 mma(float a, float b, f32x4 c) { return mfma_f32(a, b, c); }
    __device__ static int row(int g, int r) { return MathTraits<M_F32>::acc_row(g, r); }
};
template <> struct Sk<double> {
    typedef f64x4 acc;
    static constexpr int VE = 2;
    __device__ static double at(const V16 &v, int e) { return v.d[e]; }
    __device__ static void zero(V16 &v, int e) { v.d[e] = 0.0; }
    __device__ static f64x4 mma(double a, double b, f64x4 c) { return mfma_f64(a, b, c); }
    __device__ static int row(int g, int r) { return MathTraits<M_F64>::acc_row(g, r); }
};
typedef u32x4 u32x4_e __attribute__((aligned(4)));   // 16 bytes at any element
template <typename T> __device__ __forceinline__ V16 ldu(const T *p) {
    V16 v;
    v.u = *reinterpret_cast<const u32x4_e *>(p);
    return v;
}
// Zeroes the values of a group fetched `back` places before its own that lie
// before it (all of them where it has no place in the row).
template <typename T> __device__ __forceinline__ void keep_from(V16 &v, int back) {
#pragma unroll
    for (int e = 0; e < Sk<T>::VE; ++e)
        if (e < back) Sk<T>::zero(v, e);
}

// W[r][j] = sum_k X[r][k] C[j][k].  A wave owns 32 rows (two 16-row blocks)
// and JB blocks of 16 columns; slot (g, e) of group u of a pass carries
// k = k0 + (4 u + g) VE + e.
template <typename T, int JB>
__global__ void __launch_bounds__(64 * SK_WAVES) k_bwd_w(const T *__restrict__ X, const T *__restrict__ C,
                                                         T *__restrict__ W, int64_t M, int I3, int J3) {
    typedef Sk<T> K;
    constexpr int VE = K::VE, U = JB > 2 ? 2 : 4, KP = 4 * VE * U;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int64_t r0 = (int64_t(blockIdx.x) * SK_WAVES + wave) * 32;
    if (r0 >= M) return;
    const T *xr[2], *cr[JB];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        const int64_t row = r0 + mb * 16 + l16;
        xr[mb] = X + (row < M ? row : M - 1) * I3;
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {   // columns past J3 repeat the last one and are not stored
        const int j = jb * 16 + l16;
        cr[jb] = C + int64_t(j < J3 ? j : J3 - 1) * I3;
    }
    typename K::acc acc[2][JB];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) acc[mb][jb] = zero_accv<typename K::acc>();
    auto pass = [&](int k0, bool tail) __attribute__((always_inline)) {
        V16 xa[2][U], cb[JB][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + (4 * u + g) * VE, kk = tail && k > I3 - VE ? I3 - VE : k;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) xa[mb][u] = ldu(xr[mb] + kk);
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) cb[jb][u] = ldu(cr[jb] + kk);
        }
        if (tail)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int back = k0 + (4 * u + g) * VE - (I3 - VE);
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) keep_from<T>(xa[mb][u], back);
#pragma unroll
                for (int jb = 0; jb < JB; ++jb) keep_from<T>(cb[jb][u], back);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < VE; ++e)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb)
                        acc[mb][jb] = K::mma(K::at(xa[mb][u], e), K::at(cb[jb][u], e), acc[mb][jb]);
    };
    int k0 = 0;
    for (; k0 + KP <= I3; k0 += KP) pass(k0, false);
    if (k0 < I3) pass(k0, true);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int64_t row = r0 + mb * 16 + K::row(g, rr);
            if (row >= M) continue;
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
                if (jb * 16 + l16 < J3) W[row * J3 + jb * 16 + l16] = acc[mb][jb][rr];
        }
}

// part[s][j][i] = sum_{r in split s} R[r][j] X[r][i].  grid (splits,
// ceil(I3 / (64 VE))); eight waves, wave (half, cq) owning 16 VE columns i and
// half of the split's rows, the halves added through LDS in order; slot g of a
// step carries row r0 + g, column n of product e is i = i0 + VE n + e.
template <typename T, int JB>
__global__ void __launch_bounds__(512) k_bwd_dc(const T *__restrict__ R, const T *__restrict__ X, T *__restrict__ part,
                                                int64_t M, int I3, int J3, int64_t rows_per_split) {
    typedef Sk<T> K;
    constexpr int VE = K::VE, U = JB > 2 ? 4 : 8;
    __shared__ T red[4][JB * VE * 4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int cq = wave & 3, half = wave >> 2;
    const int i0 = (blockIdx.y * 4 + cq) * 16 * VE;
    const int ii = i0 + VE * l16 < I3 - VE ? i0 + VE * l16 : I3 - VE;     // first column of this lane
    const int64_t hs = (rows_per_split / 2 + 3) & ~int64_t(3);
    const int64_t sb = int64_t(blockIdx.x) * rows_per_split, se = M < sb + rows_per_split ? M : sb + rows_per_split;
    const int64_t rb = half ? sb + hs : sb, re = half ? se : (se < sb + hs ? se : sb + hs);
    typename K::acc acc[JB][VE];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int e = 0; e < VE; ++e) acc[jb][e] = zero_accv<typename K::acc>();
    int jc[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) jc[jb] = jb * 16 + l16 < J3 ? jb * 16 + l16 : J3 - 1;
    auto pass = [&](int64_t r0, bool tail) __attribute__((always_inline)) {
        V16 xb[U];
        T ra[U][JB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = r0 + 4 * u + g, rc = tail && row >= re ? re - 1 : row;
            xb[u] = ldu(X + rc * I3 + ii);
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) ra[u][jb] = R[rc * J3 + jc[jb]];
        }
        if (tail)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (r0 + 4 * u + g >= re) {
                    xb[u] = zero16();
#pragma unroll
                    for (int jb = 0; jb < JB; ++jb) ra[u][jb] = T(0);
                }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < VE; ++e)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb) acc[jb][e] = K::mma(ra[u][jb], K::at(xb[u], e), acc[jb][e]);
    };
    if (i0 < I3 && rb < re) {
        int64_t r0 = rb;
        for (; r0 + 4 * U <= re; r0 += 4 * U) pass(r0, false);
        if (r0 < re) pass(r0, true);
    }
    if (half) {
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
#pragma unroll
            for (int e = 0; e < VE; ++e)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) red[cq][(jb * VE + e) * 4 + rr][lane] = acc[jb][e][rr];
    }
    __syncthreads();
    if (half || i0 + VE * l16 >= I3) return;
    T *pp = part + int64_t(blockIdx.x) * J3 * I3;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int j = jb * 16 + K::row(g, rr);
            if (j >= J3) continue;
            V16 v;
#pragma unroll
            for (int e = 0; e < VE; ++e) {
                const T x = acc[jb][e][rr] + red[cq][(jb * VE + e) * 4 + rr][lane];
                if constexpr (VE == 4) v.f[e] = x;
                else v.d[e] = x;
            }
            *reinterpret_cast<u32x4_e *>(pp + int64_t(j) * I3 + ii) = v.u;
        }
}

// dX[r][i] = sum_j R[r][j] C[j][i].  grid (ceil(M / DX_ROWS), ceil(I3 /
// (64 VE))); a wave owns 16 VE columns i and keeps their C fragments in
// registers; slot (g, e) of group h carries j = (4 h + g) VE + e, column n of
// output product t is i = i0 + VE n + t, so each lane stores 16 bytes per row.
constexpr int DX_ROWS = 64;
template <typename T, int NH>
__global__ void __launch_bounds__(64 * SK_WAVES) k_bwd_dx(const T *__restrict__ R, const T *__restrict__ C,
                                                          T *__restrict__ dX, int64_t M, int I3, int J3) {
    typedef Sk<T> K;
    constexpr int VE = K::VE;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int i0 = (blockIdx.y * SK_WAVES + wave) * 16 * VE;
    if (i0 >= I3) return;
    const int ii = i0 + VE * l16 < I3 - VE ? i0 + VE * l16 : I3 - VE;
    const int64_t rb = int64_t(blockIdx.x) * DX_ROWS;
    const int64_t re = M < rb + DX_ROWS ? M : rb + DX_ROWS;
    int js[NH], back[NH];
    V16 cf[NH][VE];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const int j = (4 * h + g) * VE;
        js[h] = j < J3 - VE ? j : J3 - VE;
        back[h] = j - js[h];
#pragma unroll
        for (int e = 0; e < VE; ++e) {
            cf[h][e] = ldu(C + int64_t(js[h] + e) * I3 + ii);
            if (e < back[h]) cf[h][e] = zero16();
        }
    }
    auto rows = [&](int64_t r0, V16 (&ra)[NH]) __attribute__((always_inline)) {
        const int64_t row = r0 + l16 < re ? r0 + l16 : re - 1;
#pragma unroll
        for (int h = 0; h < NH; ++h) ra[h] = ldu(R + row * J3 + js[h]);
    };
    V16 cur[NH], nxt[NH];
    rows(rb, cur);
#pragma unroll
    for (int q = 0; q < DX_ROWS / 16; ++q) {
        const int64_t r0 = rb + 16 * q;
        if (r0 >= re) break;
        rows(r0 + 16, nxt);
#pragma unroll
        for (int h = 0; h < NH; ++h) keep_from<T>(cur[h], back[h]);
        typename K::acc acc[VE];
#pragma unroll
        for (int t = 0; t < VE; ++t) acc[t] = zero_accv<typename K::acc>();
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int e = 0; e < VE; ++e)
#pragma unroll
                for (int t = 0; t < VE; ++t) acc[t] = K::mma(K::at(cur[h], e), K::at(cf[h][e], t), acc[t]);
        if (i0 + VE * l16 < I3)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int64_t r = r0 + K::row(g, rr);
                if (r >= re) continue;
                V16 v;
#pragma unroll
                for (int t = 0; t < VE; ++t) {
                    if constexpr (VE == 4) v.f[t] = acc[t][rr];
                    else v.d[t] = acc[t][rr];
                }
                *reinterpret_cast<u32x4_e *>(dX + r * I3 + ii) = v.u;
            }
#pragma unroll
        for (int h = 0; h < NH; ++h) cur[h] = nxt[h];
    }
}

// V[i1][j2][j3] = sum_i2 B[j2][i2] W[i1][i2][j3] (J2, J3 <= 16 JB).  A
// workgroup owns one i1; its four waves split the i2 range and add their
// partials through LDS in order.  Slot (g, e) of a pass carries
// i2 = k0 + g VE + e: B is read 16 bytes per lane, W one value per lane (16
// consecutive j3 of a row).  Rows and columns past J repeat the last one and
// are not stored.
template <typename T, int JB>
__global__ void __launch_bounds__(64 * SK_WAVES) k_bwd_v(const T *__restrict__ B, const T *__restrict__ W, T *__restrict__ V,
                                                         int I2, int J2, int J3) {
    typedef Sk<T> K;
    constexpr int VE = K::VE, KP = 4 * VE;
    __shared__ T red[SK_WAVES - 1][JB * 4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int64_t i1 = blockIdx.x;
    const int per = ((I2 + SK_WAVES - 1) / SK_WAVES + KP - 1) / KP * KP;
    const int kb = wave * per, ke = kb + per < I2 ? kb + per : I2;
    const T *br[JB], *wc[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        const int j = jb * 16 + l16;
        br[jb] = B + int64_t(j < J2 ? j : J2 - 1) * I2;
        wc[jb] = W + i1 * I2 * J3 + (j < J3 ? j : J3 - 1);
    }
    typename K::acc acc[JB][JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int nb = 0; nb < JB; ++nb) acc[jb][nb] = zero_accv<typename K::acc>();
    for (int k0 = kb; k0 < ke; k0 += KP) {
        const int k = k0 + g * VE, kk = k < I2 - VE ? k : I2 - VE;
        V16 ba[JB];
        T wb[JB][VE];
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) ba[jb] = ldu(br[jb] + kk);
#pragma unroll
        for (int nb = 0; nb < JB; ++nb)
#pragma unroll
            for (int e = 0; e < VE; ++e) wb[nb][e] = wc[nb][int64_t(kk + e) * J3];
        if (k0 + KP > I2)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                keep_from<T>(ba[jb], k - kk);
#pragma unroll
                for (int e = 0; e < VE; ++e)
                    if (e < k - kk) wb[jb][e] = T(0);
            }
#pragma unroll
        for (int e = 0; e < VE; ++e)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int nb = 0; nb < JB; ++nb) acc[jb][nb] = K::mma(K::at(ba[jb], e), wb[nb][e], acc[jb][nb]);
    }
    // a block row at a time, so that the partials fit LDS
    T *Vp = V + i1 * J2 * J3;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        if (jb) __syncthreads();
        if (wave > 0)
#pragma unroll
            for (int nb = 0; nb < JB; ++nb)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) red[wave - 1][nb * 4 + rr][lane] = acc[jb][nb][rr];
        __syncthreads();
        if (wave == 0)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int j2 = jb * 16 + K::row(g, rr);
#pragma unroll
                for (int nb = 0; nb < JB; ++nb) {
                    T x = acc[jb][nb][rr];
#pragma unroll
                    for (int w = 0; w < SK_WAVES - 1; ++w) x += red[w][nb * 4 + rr][lane];
                    if (j2 < J2 && nb * 16 + l16 < J3) Vp[j2 * J3 + nb * 16 + l16] = x;
                }
            }
    }
}

// R[i1][i2][j3] = sum_j2 B[j2][i2] H[i1][j2][j3] (J3 <= 16 JB).  A wave owns 32
// rows i2 of one i1 (grid (I1, ceil(I2 / 128))); slot g of step u of a pass
// carries j2 = 4 (s + u) + g; B and H are read one value per lane (16
// consecutive i2 or j3), R written 16 values per row and 16 lanes.
template <typename T, int JB>
__global__ void __launch_bounds__(64 * SK_WAVES) k_bwd_r(const T *__restrict__ B, const T *__restrict__ H, T *__restrict__ R,
                                                         int I2, int J2, int J3) {
    typedef Sk<T> K;
    constexpr int U = 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int64_t i1 = blockIdx.x;
    const int m0 = (blockIdx.y * SK_WAVES + wave) * 32;
    if (m0 >= I2) return;
    const T *Hp = H + i1 * J2 * J3;
    int ic[2], jc[JB];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) ic[mb] = m0 + 16 * mb + l16 < I2 ? m0 + 16 * mb + l16 : I2 - 1;
#pragma unroll
    for (int nb = 0; nb < JB; ++nb) jc[nb] = nb * 16 + l16 < J3 ? nb * 16 + l16 : J3 - 1;
    typename K::acc acc[2][JB];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < JB; ++nb) acc[mb][nb] = zero_accv<typename K::acc>();
    for (int s = 0; s < J2; s += 4 * U) {
        T a[U][2], h[U][JB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j2 = s + 4 * u + g, jj = j2 < J2 ? j2 : J2 - 1;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) a[u][mb] = B[int64_t(jj) * I2 + ic[mb]];
#pragma unroll
            for (int nb = 0; nb < JB; ++nb) h[u][nb] = Hp[jj * J3 + jc[nb]];
        }
        if (s + 4 * U > J2)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s + 4 * u + g >= J2) {
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) a[u][mb] = T(0);
#pragma unroll
                    for (int nb = 0; nb < JB; ++nb) h[u][nb] = T(0);
                }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < JB; ++nb) acc[mb][nb] = K::mma(a[u][mb], h[u][nb], acc[mb][nb]);
    }
    T *Rp = R + i1 * int64_t(I2) * J3;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int i2 = m0 + 16 * mb + K::row(g, rr);
            if (i2 >= I2) continue;
#pragma unroll
            for (int nb = 0; nb < JB; ++nb)
                if (nb * 16 + l16 < J3) Rp[int64_t(i2) * J3 + nb * 16 + l16] = acc[mb][nb][rr];
        }
}

// out[e] = sum_{s < S} part[s n + e] of up to three split products in one
// launch.  A workgroup owns 64 elements; its four waves each sum a quarter of
// the partials in order with eight loads in flight, and the quarters are added
// in order.  (One launch per product, two where there were more than sixteen
// partials, took 4.5 us each whatever their size.)
template <typename T> struct SumArgs {
    const T *part[3];
    T *out[3];
    int64_t n[3];
    int S[3];
    int64_t first[3];   // first workgroup of each
};
template <typename T>
__global__ void __launch_bounds__(256) k_bwd_sum(const SumArgs<T> a, int count) {
    __shared__ T red[3][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int w = 0;
    while (w + 1 < count && int64_t(blockIdx.x) >= a.first[w + 1]) ++w;
    const int64_t n = a.n[w], e = (int64_t(blockIdx.x) - a.first[w]) * 64 + lane;
    const int per = (a.S[w] + 3) / 4, sb = wave * per, se = sb + per < a.S[w] ? sb + per : a.S[w];
    const T *p = a.part[w] + (e < n ? e : n - 1);
    T acc = T(0);
    int s = sb;
    for (; s + 8 <= se; s += 8) {
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(s + u) * n];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; s < se; ++s) acc += p[s * n];
    if (wave) red[wave - 1][lane] = acc;
    __syncthreads();
    if (wave == 0 && e < n) a.out[w][e] = ((acc + red[0][lane]) + red[1][lane]) + red[2][lane];
}

// ---------------------------------------------------------------------------
// Fused adjoint for float32 with J1, J2, J3 <= 32, I3 in {256, 512} and I2 a
// multiple of 4: two launches in place of the product sequence above.
//
//   k_bwd_xpass_f32    one workgroup per slab X[i1] reads the slab once and
//                      writes dX[i1] once.  With H = G x1 A^T formed in the
//                      workgroup and R = H x2 B^T formed per chunk of rows,
//                      each chunk of X is contracted twice on the matrix cores
//                      (with C for the rows of W = X x3 C, with R for the
//                      slab's share of dC), and dX = R x3 C^T is written for
//                      the same rows.  W never leaves the chip: each chunk of
//                      its rows is contracted with B (the slab's V = X x2 B x3
//                      C) and with H (the slab's columns of its dB share); at
//                      the end dA[:, i1] = G_(1) vec(V).
//   k_bwd_finish_f32   dB and dC as fixed-order sums of the slabs' shares.
//
// The slab streams through LDS in chunks of CR rows x I3 (32 KiB): three
// stages filled by direct-to-LDS copies two chunks ahead, with B's matching
// CR columns in four stages, so that every global read in the loop is a copy
// the kernel waits for explicitly.  Wave (rh, cq) owns row block rh (16 rows)
// and column group cq (64 columns) of each chunk; it reads its 16 x 64 block
// twice: in the W product a lane holds row l % 16 and four consecutive
// columns (the k slots), in the dC product row l / 16 of a k step (the k
// slot) and four consecutive columns (the output columns of four products).
// X words are XOR-swizzled by the row's low four bits so that both reads
// cover all banks.  The W partials of the column groups meet in LDS; their
// V and dB work, and the R of the chunk after next, run in the following
// iteration ahead of its products (double-buffered W partials and R), so one
// barrier per chunk orders everything.  Padded factor rows (j >= J) are
// zeros; rows past I2 read the last row and are masked where they contribute.
// ---------------------------------------------------------------------------
constexpr int FB_THREADS = 512;
constexpr int FB_XSTAGE = 32768;   // bytes of one X chunk

struct FusedArgs {
    const float *X, *A, *B, *C, *G;
    float *partB, *partC;           // workspace: I1 x J2 x I2, I1 x J3 x I3
    float *dX, *dA, *dB, *dC;
    int64_t I1;
    int I2, I3, J1, J2, J3;
    int nbB, nbC;                   // finish kernel: blocks of dB and dC sums
};

template <int NCG>
__global__ void __launch_bounds__(FB_THREADS, 1) k_bwd_xpass_f32(const FusedArgs a) {
    constexpr int NRG = 8 / NCG;                 // 16-row blocks per chunk
    constexpr int CR = 16 * NRG;                 // rows per chunk
    constexpr int I3C = 64 * NCG;
    constexpr int WPR = I3C / 4;                 // 16-byte words per X row
    constexpr int XOPS = FB_XSTAGE / 1024 / 8;   // 16-byte copies per wave per chunk
    constexpr int BSTAGE = 32 * CR * 4;          // bytes of B's chunk: 32 rows j2 x CR columns
    constexpr int BOPS = BSTAGE / 256 / 8;       // 4-byte copies per wave per chunk
    constexpr int WPS = 16 * 33;                 // one wave's W partial tile (padded rows)
    static_assert(NCG == 4 || NCG == 8, "four or eight 64-column groups");
    static_assert(XOPS < 16, "vmcnt range");
    static_assert(32 * FB_THREADS * 4 <= 3 * FB_XSTAGE && 32 * 16 * 4 <= 4 * BSTAGE, "reduction space");

    __shared__ __align__(1024) unsigned char xbuf[3 * FB_XSTAGE];
    __shared__ __align__(256) float bbuf[4][32 * CR];
    __shared__ float rbuf[2][CR * 36];          // R rows padded to 36 floats
    __shared__ float wpart[2][NRG * NCG * WPS];
    __shared__ float hbuf[32 * 33];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rh = wave / NCG, cq = wave % NCG;
    const int h = lane & 15, g = lane >> 4;
    const int64_t i1 = blockIdx.x;
    const int I2 = a.I2, J2 = a.J2, J3 = a.J3;
    const int nch = (I2 + CR - 1) / CR;
    const float *Xs = a.X + i1 * int64_t(I2) * I3C;
    const uint32_t xlds = lds_offset(xbuf), blds = lds_offset(&bbuf[0][0]);

    // chunk c of X into stage c % 3: LDS word q of the stage is row q / WPR,
    // position q % WPR, holding the row's word (q % WPR) ^ (row & 15)
    auto issue_x = [&](int c) __attribute__((always_inline)) {
        const uint32_t st = xlds + uint32_t((c % 3) * FB_XSTAGE);
#pragma unroll
        for (int j = 0; j < XOPS; ++j) {
            const int q = (wave * XOPS + j) * 64 + lane, row = q / WPR, pw = q % WPR;
            const int gr = c * CR + row < I2 ? c * CR + row : I2 - 1;
            dma16_to_lds_m0(Xs + int64_t(gr) * I3C + 4 * (pw ^ (row & 15)), st + uint32_t((wave * XOPS + j) * 1024));
        }
    };
    // B[:, chunk c] into stage c % 4: float p of row j2 holds column
    // c CR + (p ^ bsw(j2)), spreading the 16 rows a fragment read touches
    auto bsw = [](int j2) __attribute__((always_inline)) { return ((j2 * CR) >> 6) & (CR - 1); };
    auto issue_b = [&](int c) __attribute__((always_inline)) {
        const uint32_t st = blds + uint32_t((c & 3) * BSTAGE);
#pragma unroll
        for (int j = 0; j < BOPS; ++j) {
            const int f = (wave * BOPS + j) * 64 + lane, j2 = f / CR, p = f % CR;
            const int col = c * CR + (p ^ bsw(j2));
            const int j2c = j2 < J2 ? j2 : J2 - 1;
            dma4_to_lds_m0(a.B + int64_t(j2c) * I2 + (col < I2 ? col : I2 - 1), st + uint32_t((wave * BOPS + j) * 256));
        }
    };

    // copies of the first chunks, then H[i1] = sum_j1 A[j1][i1] G[j1]
    // (zero-padded to 32 x 32, to LDS and to the workspace for the dX kernel;
    // rows j1 >= J1 read row J1 - 1 with weight zero, so every load is issued
    // before the sums) and the C fragments of the W product
    issue_b(0);
    if (nch > 1) issue_b(1);
    issue_x(0);
    if (nch > 1) issue_x(1);
    {
        const int j3 = tid & 31, j2a = tid >> 5, j2b = j2a + 16;
        const bool va = j2a < J2 && j3 < J3, vb = j2b < J2 && j3 < J3;
        const int64_t gs = int64_t(J2) * J3;
        const float *ga = a.G + (va ? j2a * J3 + j3 : 0), *gb = a.G + (vb ? j2b * J3 + j3 : 0);
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int j1 = 0; j1 < 32; ++j1) {
            const int j1c = j1 < a.J1 ? j1 : a.J1 - 1;
            const float w = j1 < a.J1 ? a.A[int64_t(j1c) * a.I1 + i1] : 0.f;
            s0 += w * ga[j1c * gs];
            s1 += w * gb[j1c * gs];
        }
        s0 = va ? s0 : 0.f;
        s1 = vb ? s1 : 0.f;
        hbuf[j2a * 33 + j3] = s0;
        hbuf[j2b * 33 + j3] = s1;
    }
    // k slot (l/16, e) of step k is column 64 cq + 16 k + 4 (l/16) + e,
    // output column j3 = 16 jb + l % 16
    V16 cf[2][4];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = 16 * jb + h;
            cf[jb][k] = ld16(a.C + int64_t(j < J3 ? j : J3 - 1) * I3C + 64 * cq + 16 * k + 4 * g);
            if (j >= J3) cf[jb][k] = zero16();
        }
    // dX product: k slot (l/16, e) of half hh is j3 = 16 hh + 4 (l/16) + e,
    // column n of product t is i3 = 64 cq + 4 n + t
    V16 cfx[2][4];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = 16 * hh + 4 * g + e;
            cfx[hh][e] = ld16(a.C + int64_t(j < J3 ? j : J3 - 1) * I3C + 64 * cq + 4 * h);
            if (j >= J3) cfx[hh][e] = zero16();
        }
    wait_vmcnt<0>();
    __syncthreads();

    // Each wave's share of the work on a chunk's W partials: V piece v =
    // wave (tile v / NRG, row block v % NRG) when v < 4 NRG, and task t:
    // dB tile t (columns 16 (t / NRG).., row block t % NRG) for t < 2 NRG, R
    // tile t - 2 NRG (row block (t - 2 NRG) / 2, columns 16 ((t - 2 NRG) & 1)..)
    // for t < 4 NRG.  Its H operand: hs[k] = H[16 jb2 + l%16][4 k + l/16] for
    // a dB tile, H[4 k + l/16][16 jb3 + l%16] for an R tile.
    const int task = NRG == 1 ? (wave + 4) & 7 : wave;
    const bool has_v = wave < 4 * NRG, is_db = task < 2 * NRG, is_r = !is_db && task < 4 * NRG;
    const int v_t = wave / NRG, v_rb = wave % NRG;
    const int db_jb2 = task / NRG, db_rb = task % NRG;
    const int r_rb = (task - 2 * NRG) >> 1, r_jb3 = (task - 2 * NRG) & 1;
    float hs[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        hs[k] = is_db ? hbuf[(16 * db_jb2 + h) * 33 + 4 * k + g]
                      : (is_r ? hbuf[(4 * k + g) * 33 + 16 * r_jb3 + h] : 0.f);

    f32x4 dcacc[2][4], vacc = zero_accv<f32x4>(), dbt = zero_accv<f32x4>(), dxa[4];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int e = 0; e < 4; ++e) dcacc[jb][e] = zero_accv<f32x4>();
    float *pb = a.partB + i1 * int64_t(J2) * I2;

    // R of chunk cn (rows past I2 zero) into rbuf[cn & 1]
    auto r_tiles = [&](int cn) __attribute__((always_inline)) {
        if (!is_r) return;
        const float *bn = bbuf[cn & 3];
        f32x4 acc = zero_accv<f32x4>();
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int j2 = 4 * k + g, rho = 16 * r_rb + h;
            acc = mfma_f32(bn[j2 * CR + (rho ^ bsw(j2))], hs[k], acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rho = 16 * r_rb + 4 * g + r;
            rbuf[cn & 1][rho * 36 + 16 * r_jb3 + h] = cn * CR + rho < I2 ? acc[r] : 0.f;
        }
    };
    // V and dB of chunk cp from its summed W partials
    auto w_work = [&](int cp) __attribute__((always_inline)) {
        const float *bs = bbuf[cp & 3];
        const float *wp = wpart[cp & 1];
        if (has_v) {
            const int jb2 = v_t >> 1, jb3 = v_t & 1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // V[j2][j3] += sum_rows B[j2][row] W[row][j3]
                const int rho = 16 * v_rb + 4 * k + g, j2 = 16 * jb2 + h;
                float av = bs[j2 * CR + (rho ^ bsw(j2))];
                if (cp * CR + rho >= I2) av = 0.f;
                float bv = 0.f;
#pragma unroll
                for (int q = 0; q < NCG; ++q) bv += wp[(v_rb * NCG + q) * WPS + (4 * k + g) * 33 + 16 * jb3 + h];
                vacc = mfma_f32(av, bv, vacc);
            }
        }
        if (is_db) {
            // dB[j2][row] = sum_j3 H[j2][j3] W[row][j3]
            f32x4 acc = zero_accv<f32x4>();
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float bv = 0.f;
#pragma unroll
                for (int q = 0; q < NCG; ++q) bv += wp[(db_rb * NCG + q) * WPS + h * 33 + 4 * k + g];
                acc = mfma_f32(hs[k], bv, acc);
            }
            dbt = acc;
        }
    };
    // stores of results kept in registers: a chunk's dB tile and dX block
    auto store_db = [&](int cp) __attribute__((always_inline)) {
        if (!is_db) return;
        const int col = cp * CR + 16 * db_rb + h;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j2 = 16 * db_jb2 + 4 * g + r;
            if (j2 < J2 && col < I2) pb[int64_t(j2) * I2 + col] = dbt[r];
        }
    };
    float *dXs = a.dX ? a.dX + i1 * int64_t(I2) * I3C + 64 * cq + 4 * h : nullptr;
    auto store_dx = [&](int cp) __attribute__((always_inline)) {
        if (!dXs) return;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = cp * CR + 16 * rh + 4 * g + r;
            const f32x4 v = {dxa[0][r], dxa[1][r], dxa[2][r], dxa[3][r]};
            if (row < I2) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(dXs + int64_t(row) * I3C));
        }
    };

    r_tiles(0);
    for (int c = 0; c < nch; ++c) {
        // X(c) and B(c + 1) have landed when at most the X copies issued in
        // iteration c - 1 (the last copies, after its B copies) are
        // outstanding; stores issued after them only make the wait longer
        if (c + 1 < nch) wait_vmcnt<XOPS>();
        else wait_vmcnt<0>();
        __syncthreads();
        // the previous iterations' results go out ahead of this iteration's
        // copies, so that the next wait finds them older than the copies
        if (c > 0) store_dx(c - 1);
        if (c > 1) store_db(c - 2);
        if (c + 2 < nch) {
            issue_b(c + 2);
            issue_x(c + 2);
        }
        // the previous chunk's W work and the next chunk's R run ahead of
        // this chunk's products (different buffers; the barrier above orders
        // them against both)
        if (c > 0) w_work(c - 1);
        if (c + 1 < nch) r_tiles(c + 1);

        // products on this wave's 16 x 64 block of the chunk
        const float *xs = reinterpret_cast<const float *>(xbuf + (c % 3) * FB_XSTAGE);
        const float *rs = rbuf[c & 1];
        f32x4 wacc[2][2];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) wacc[jb][0] = wacc[jb][1] = zero_accv<f32x4>();
        // dC: k slot = row 16 rh + 4 k + l/16, product e takes column 64 cq + 4 (l%16) + e;
        // W: row 16 rh + l%16, k slot (l/16, e) = column 64 cq + 16 k + 4 (l/16) + e
        const float *xrow_c = xs + (16 * rh + g) * I3C + 64 * cq;
        const float *xrow_w = xs + (16 * rh + h) * I3C + 64 * cq + 4 * (g ^ (h & 3));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            V16 xv, xw;
            xv.u = *reinterpret_cast<const u32x4 *>(xrow_c + 4 * k * I3C + 4 * (h ^ (4 * k + g)));
            xw.u = *reinterpret_cast<const u32x4 *>(xrow_w + 16 * (k ^ (h >> 2)));
            const int rr = 16 * rh + 4 * k + g;
            const float r0 = rs[rr * 36 + h], r1 = rs[rr * 36 + 16 + h];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dcacc[0][e] = mfma_f32(r0, xv.f[e], dcacc[0][e]);
                dcacc[1][e] = mfma_f32(r1, xv.f[e], dcacc[1][e]);
                wacc[0][k & 1] = mfma_f32(xw.f[e], cf[0][k].f[e], wacc[0][k & 1]);
                wacc[1][k & 1] = mfma_f32(xw.f[e], cf[1][k].f[e], wacc[1][k & 1]);
            }
        }
        float *wp = wpart[c & 1] + (rh * NCG + cq) * WPS;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) wp[(4 * g + r) * 33 + 16 * jb + h] = wacc[jb][0][r] + wacc[jb][1][r];
        // dX[row][i3] = sum_j3 R[row][j3] C[j3][i3] for this wave's block
        if (dXs) {
#pragma unroll
            for (int t = 0; t < 4; ++t) dxa[t] = zero_accv<f32x4>();
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                V16 ra;
                ra.u = *reinterpret_cast<const u32x4 *>(rs + (16 * rh + h) * 36 + 16 * hh + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int t = 0; t < 4; ++t) dxa[t] = mfma_f32(ra.f[e], cfx[hh][e].f[t], dxa[t]);
            }
        }
    }
    store_dx(nch - 1);
    if (nch > 1) store_db(nch - 2);
    __syncthreads();
    w_work(nch - 1);
    store_db(nch - 1);

    // the row blocks' dC shares and the V pieces are added through LDS in a
    // fixed order (no copy is outstanding: the stages are free)
    __syncthreads();
    float *red = reinterpret_cast<float *>(xbuf);
    float *vred = red + (NRG - 1) * NCG * 2048;
    if (rh > 0) {
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    red[((rh - 1) * NCG + cq) * 2048 + ((jb * 4 + e) * 4 + r) * 64 + lane] = dcacc[jb][e][r];
    }
    if (has_v)
#pragma unroll
        for (int r = 0; r < 4; ++r) vred[(wave * 4 + r) * 64 + lane] = vacc[r];
    __syncthreads();
    if (rh == 0) {
        for (int q = 1; q < NRG; ++q)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        dcacc[jb][e][r] += red[((q - 1) * NCG + cq) * 2048 + ((jb * 4 + e) * 4 + r) * 64 + lane];
        float *pc = a.partC + i1 * int64_t(J3) * I3C;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j3 = 16 * jb + 4 * g + r;
                if (j3 >= J3) continue;
                const f32x4 v = {dcacc[jb][0][r], dcacc[jb][1][r], dcacc[jb][2][r], dcacc[jb][3][r]};
                *reinterpret_cast<f32x4 *>(pc + int64_t(j3) * I3C + 64 * cq + 4 * h) = v;
            }
    }
    if (!a.dA) return;
    // V[i1] (32 x 32, padded) into hbuf
    if (wave < 4) {
        const int jb2 = wave >> 1, jb3 = wave & 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float s = 0.f;
            for (int rb = 0; rb < NRG; ++rb) s += vred[((wave * NRG + rb) * 4 + r) * 64 + lane];
            hbuf[(16 * jb2 + 4 * g + r) * 33 + 16 * jb3 + h] = s;
        }
    }
    __syncthreads();
    // dA[j1][i1] = sum_n G[j1][n] V[i1][n], n = j2 J3 + j3: thread t takes
    // n = t and t + 512 (coalesced rows of G) for every j1; the 512 partial
    // sums of each j1 are then added in thread order, sixteen runs of 32 and
    // then the sixteen run sums
    {
        const int NN = J2 * J3;
        float vv[2];
        int nn[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int n = tid + FB_THREADS * m;
            const bool ok = n < NN;
            nn[m] = ok ? n : 0;
            vv[m] = ok ? hbuf[(n / J3) * 33 + n % J3] : 0.f;
        }
        float *red2 = reinterpret_cast<float *>(xbuf);   // [32 j1][512 threads], after the dC shares were read
        float *red3 = &bbuf[0][0];                      // [32 j1][16 runs]
#pragma unroll
        for (int j1 = 0; j1 < 32; ++j1) {
            const float *gr = a.G + int64_t(j1 < a.J1 ? j1 : a.J1 - 1) * NN;
            red2[j1 * FB_THREADS + tid] = gr[nn[0]] * vv[0] + gr[nn[1]] * vv[1];
        }
        __syncthreads();
        {
            const int j1 = tid >> 4, run = tid & 15;
            float s = 0.f;
            for (int q = 0; q < 32; ++q) s += red2[j1 * FB_THREADS + run * 32 + q];
            red3[j1 * 16 + run] = s;
        }
        __syncthreads();
        if (tid < a.J1) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) s += red3[tid * 16 + q];
            a.dA[int64_t(tid) * a.I1 + i1] = s;
        }
    }
}

// Blocks [0, nbB) and [nbB, nbB + nbC): 64 consecutive elements of dB (or
// dC) each, the sum over i1 of the slabs' shares: 16 groups of consecutive
// i1, each summed in increasing i1 by one thread per 4 elements, then the 16
// group sums in increasing group order.
__global__ void __launch_bounds__(256) k_bwd_finish_f32(const FusedArgs a) {
    __shared__ f32x4 red[16][16];
    const int tid = threadIdx.x, b = blockIdx.x;
    const bool isB = b < a.nbB;
    const int64_t n = isB ? int64_t(a.J2) * a.I2 : int64_t(a.J3) * a.I3;
    const float *part = isB ? a.partB : a.partC;
    float *out = isB ? a.dB : a.dC;
    const int f = tid & 15, grp = tid >> 4;
    const int64_t e4 = (int64_t(isB ? b : b - a.nbB) * 16 + f) * 4;
    const int64_t gs = (a.I1 + 15) / 16, lo = grp * gs, hi = lo + gs < a.I1 ? lo + gs : a.I1;
    f32x4 s = zero_accv<f32x4>();
    if (e4 < n)
        for (int64_t i0 = lo; i0 < hi; i0 += 16) {
            // sixteen loads in flight, added in increasing i1
            f32x4 v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                v[u] = *reinterpret_cast<const f32x4 *>(part + (i0 + u < hi ? i0 + u : lo) * n + e4);
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (i0 + u < hi) s += v[u];
        }
    red[grp][f] = s;
    __syncthreads();
    if (tid < 16 && e4 < n) {
        f32x4 t = zero_accv<f32x4>();
#pragma unroll
        for (int q = 0; q < 16; ++q) t += red[q][tid];
        *reinterpret_cast<f32x4 *>(out + e4) = t;
    }
}

// The split products whose partials the call's last launch sums.
template <typename T>
struct Sums {
    SumArgs<T> a;
    int count = 0;
    int64_t groups = 0;
    void add(const void *part, void *out, int64_t n, int S) {
        a.part[count] = static_cast<const T *>(part);
        a.out[count] = static_cast<T *>(out);
        a.n[count] = n;
        a.S[count] = S;
        a.first[count++] = groups;
        groups += ceil_div(n, 64);
    }
    int run(hipStream_t st) const {
        if (!count) return TTM_OK;
        return launch("ttm_bwd_sum_splits", st, [&] {
            hipLaunchKernelGGL(k_bwd_sum<T>, dim3(unsigned(groups)), dim3(256), 0, st, a, count);
        });
    }
};

// split: null, or where the partials of a split k range are to be summed
template <int MATH>
int run_gemm(GemmArgs a, int64_t batch, Sums<typename MathTraits<MATH>::acc_t> *split, void *part, hipStream_t st,
             const char *name) {
    typedef typename MathTraits<MATH>::acc_t T;
    const int64_t KT = GemmCfg<MATH>::KT;
    if (a.Ki <= 0) a.Ki = a.K;
    SplitK k = split ? choose_split(a.M, a.N, a.K, batch, KT) : SplitK{1, round_up(a.K, KT)};
    void *final_out = a.C;
    if (k.ks > 1) {
        // partials are dense row-major M x N (batch must be 1 here)
        a.C = part;
        a.scm = a.N;
        a.scn = 1;
        a.scs = a.M * a.N;
    }
    a.k_per_split = k.per;
    // 16-byte operand loads along the unit-stride dimension where every
    // group of VG elements stays inside the extent, the k split and one
    // address-aligned run
    {
        const int64_t VG = int64_t(16 / sizeof(T));
        const bool kk = a.K % VG == 0 && a.Ki % VG == 0 && a.k_per_split % VG == 0;
        auto vec_ok = [&](const void *ptr, int64_t sfast_m, int64_t sk, int64_t sko, int64_t sb, int64_t sp,
                          int64_t extent) -> int {
            if (!aligned(ptr, 16) || sb % VG || sp % VG) return 0;
            if (sk == 1) return (kk && sfast_m % VG == 0 && (a.Ki == a.K || sko % VG == 0)) ? 1 : 0;
            if (sfast_m == 1) return (extent % VG == 0 && sk % VG == 0 && (a.Ki == a.K || sko % VG == 0)) ? 1 : 0;
            return 0;
        };
        a.vec_a = vec_ok(a.A, a.sam, a.saki, a.sako, a.sab, 0, a.M);
        a.vec_b = vec_ok(a.B, a.sbn, a.sbki, a.sbko, a.sbb, a.P > 1 ? a.sbp : 0, a.N);
    }
    dim3 grid(unsigned(ceil_div(a.M, 64) * ceil_div(a.N, 64)), unsigned(k.ks), unsigned(batch));
    int rc = launch(name, st, [&] {
        if (a.vec_a && a.vec_b) hipLaunchKernelGGL((k_gemm<MATH, true, true>), grid, dim3(256), 0, st, a);
        else if (a.vec_a) hipLaunchKernelGGL((k_gemm<MATH, true, false>), grid, dim3(256), 0, st, a);
        else if (a.vec_b) hipLaunchKernelGGL((k_gemm<MATH, false, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_gemm<MATH, false, false>), grid, dim3(256), 0, st, a);
    });
    if (rc || k.ks == 1) return rc;
    split->add(part, final_out, a.M * a.N, k.ks);
    return rc;
}

template <int NCG>
int run_fused_ncg(const FusedArgs &fa, hipStream_t st) {
    int rc = launch("ttm_bwd_xpass", st, [&] {
        hipLaunchKernelGGL(k_bwd_xpass_f32<NCG>, dim3(unsigned(fa.I1)), dim3(FB_THREADS), 0, st, fa);
    });
    if (rc || fa.nbB + fa.nbC == 0) return rc;
    return launch("ttm_bwd_finish", st, [&] {
        hipLaunchKernelGGL(k_bwd_finish_f32, dim3(unsigned(fa.nbB + fa.nbC)), dim3(256), 0, st, fa);
    });
}

int run_fused(const BwdPlan &p, const void *G, const void *X, const void *A, const void *B, const void *C, void *dX,
              void *dA, void *dB, void *dC, unsigned char *ws, hipStream_t st) {
    FusedArgs fa;
    memset(&fa, 0, sizeof fa);
    fa.X = static_cast<const float *>(X);
    fa.A = static_cast<const float *>(A);
    fa.B = static_cast<const float *>(B);
    fa.C = static_cast<const float *>(C);
    fa.G = static_cast<const float *>(G);
    fa.partB = reinterpret_cast<float *>(ws + p.f_off_B);
    fa.partC = reinterpret_cast<float *>(ws + p.f_off_C);
    fa.dX = static_cast<float *>(dX);
    fa.dA = static_cast<float *>(dA);
    fa.dB = static_cast<float *>(dB);
    fa.dC = static_cast<float *>(dC);
    fa.I1 = p.I1;
    fa.I2 = int(p.I2); fa.I3 = int(p.I3);
    fa.J1 = int(p.J1); fa.J2 = int(p.J2); fa.J3 = int(p.J3);
    fa.nbB = dB ? int(ceil_div(p.J2 * p.I2, 64)) : 0;
    fa.nbC = dC ? int(ceil_div(p.J3 * p.I3, 64)) : 0;
    switch (p.ncg) {
        case 4: return run_fused_ncg<4>(fa, st);
        case 8: return run_fused_ncg<8>(fa, st);
        default: return TTM_ERR_UNSUPPORTED;
    }
}

template <int MATH>
int run_backward(const BwdPlan &p, const void *G, const void *X, const void *A, const void *B, const void *C,
                 void *dX, void *dA, void *dB, void *dC, unsigned char *ws, hipStream_t st) {
    typedef typename MathTraits<MATH>::acc_t T;
    constexpr int VE = Sk<T>::VE;
    void *W = ws + p.off_W, *V = ws + p.off_V, *H = ws + p.off_H, *R = ws + p.off_R;
    const int64_t I1 = p.I1, I2 = p.I2, I3 = p.I3, J1 = p.J1, J2 = p.J2, J3 = p.J3, NN = p.NN, M = I1 * I2;
    const T *Xt = static_cast<const T *>(X), *Bt = static_cast<const T *>(B), *Ct = static_cast<const T *>(C);
    T *Wt = static_cast<T *>(W), *Vt = static_cast<T *>(V), *Ht = static_cast<T *>(H), *Rt = static_cast<T *>(R);
    const int j3b = int(ceil_div(J3, 16));
    const dim3 sk(64 * SK_WAVES);
    Sums<T> sums;
    int rc = TTM_OK;
    if (p.need_w) {   // W[(i1,i2)][j3] = sum_i3 X[(i1,i2)][i3] C[j3][i3]
        if (p.stream) {
            const dim3 grid(unsigned(ceil_div(M, 32 * SK_WAVES)));
            rc = launch("ttm_bwd_W", st, [&] {
                auto go = [&](auto k) { hipLaunchKernelGGL(k, grid, sk, 0, st, Xt, Ct, Wt, M, int(I3), int(J3)); };
                if (j3b == 1) go(k_bwd_w<T, 1>);
                else if (j3b == 2) go(k_bwd_w<T, 2>);
                else if (j3b == 3) go(k_bwd_w<T, 3>);
                else go(k_bwd_w<T, 4>);
            });
        } else {
            GemmArgs a = gargs();
            a.A = X; a.B = C; a.C = W;
            a.M = M; a.N = J3; a.K = I3;
            a.sam = I3; a.saki = 1;
            a.sbn = I3; a.sbki = 1;
            a.scm = J3; a.scn = 1;
            rc = run_gemm<MATH>(a, 1, nullptr, nullptr, st, "ttm_bwd_W");
        }
        if (rc) return rc;
    }
    if (p.need_v) {   // V[i1][j2][j3] = sum_i2 B[j2][i2] W[i1][i2][j3]
        if (p.stream_vr) {
            rc = launch("ttm_bwd_V", st, [&] {
                auto go = [&](auto k) {
                    hipLaunchKernelGGL(k, dim3(unsigned(I1)), sk, 0, st, Bt, Wt, Vt, int(I2), int(J2), int(J3));
                };
                if (J2 <= 32 && J3 <= 32) go(k_bwd_v<T, 2>);
                else go(k_bwd_v<T, 4>);
            });
        } else {
            GemmArgs a = gargs();
            a.A = B; a.B = W; a.C = V;
            a.M = J2; a.N = J3; a.K = I2;
            a.sam = I2; a.saki = 1;
            a.sbb = I2 * J3; a.sbki = J3; a.sbn = 1;
            a.scb = NN; a.scm = J3; a.scn = 1;
            rc = run_gemm<MATH>(a, I1, nullptr, nullptr, st, "ttm_bwd_V");
        }
        if (rc) return rc;
    }
    if (dA) {         // dA[j1][i1] = sum_n G[j1][n] V[i1][n]
        GemmArgs a = gargs();
        a.A = G; a.B = V; a.C = dA;
        a.M = J1; a.N = I1; a.K = NN;
        a.sam = NN; a.saki = 1;
        a.sbn = NN; a.sbki = 1;
        a.scm = I1; a.scn = 1;
        if ((rc = run_gemm<MATH>(a, 1, &sums, ws + p.off_P[0], st, "ttm_bwd_dA"))) return rc;
    }
    if (p.need_h) {   // H[i1][n] = sum_j1 A[j1][i1] G[j1][n]
        GemmArgs a = gargs();
        a.A = A; a.B = G; a.C = H;
        a.M = I1; a.N = NN; a.K = J1;
        a.sam = 1; a.saki = I1;
        a.sbn = 1; a.sbki = NN;
        a.scm = NN; a.scn = 1;
        if ((rc = run_gemm<MATH>(a, 1, nullptr, nullptr, st, "ttm_bwd_H"))) return rc;
    }
    if (p.need_r) {   // R[i1][i2][j3] = sum_j2 B[j2][i2] H[i1][j2][j3]
        if (p.stream_vr) {
            const dim3 grid(unsigned(I1), unsigned(ceil_div(I2, 32 * SK_WAVES)));
            rc = launch("ttm_bwd_R", st, [&] {
                auto go = [&](auto k) { hipLaunchKernelGGL(k, grid, sk, 0, st, Bt, Ht, Rt, int(I2), int(J2), int(J3)); };
                if (j3b <= 2) go(k_bwd_r<T, 2>);
                else go(k_bwd_r<T, 4>);
            });
        } else {
            GemmArgs a = gargs();
            a.A = B; a.B = H; a.C = R;
            a.M = I2; a.N = J3; a.K = J2;
            a.sam = 1; a.saki = I2;
            a.sbb = NN; a.sbki = J3; a.sbn = 1;
            a.scb = I2 * J3; a.scm = J3; a.scn = 1;
            rc = run_gemm<MATH>(a, I1, nullptr, nullptr, st, "ttm_bwd_R");
        }
        if (rc) return rc;
    }
    if (dX) {         // dX[(i1,i2)][i3] = sum_j3 R[(i1,i2)][j3] C[j3][i3]
        if (p.stream) {
            const dim3 grid(unsigned(ceil_div(M, DX_ROWS)), unsigned(ceil_div(I3, 16 * VE * SK_WAVES)));
            rc = launch("ttm_bwd_dX", st, [&] {
                auto go = [&](auto k) {
                    hipLaunchKernelGGL(k, grid, sk, 0, st, Rt, Ct, static_cast<T *>(dX), M, int(I3), int(J3));
                };
                const int nh = int(ceil_div(J3, 4 * VE));   // groups of 4 VE values of j3
                constexpr int F = 4 / VE;                   // 1 (float) or 2 (double)
                if (nh <= F) go(k_bwd_dx<T, F>);
                else if (nh <= 2 * F) go(k_bwd_dx<T, 2 * F>);
                else if (nh <= 3 * F) go(k_bwd_dx<T, 3 * F>);
                else go(k_bwd_dx<T, 4 * F>);
            });
        } else {
            GemmArgs a = gargs();
            a.A = R; a.B = C; a.C = dX;
            a.M = M; a.N = I3; a.K = J3;
            a.sam = J3; a.saki = 1;
            a.sbn = 1; a.sbki = I3;
            a.scm = I3; a.scn = 1;
            rc = run_gemm<MATH>(a, 1, nullptr, nullptr, st, "ttm_bwd_dX");
        }
        if (rc) return rc;
    }
    if (dB) {         // dB[j2][i2] = sum_{i1,j3} H[i1][j2][j3] W[i1][i2][j3]
        GemmArgs a = gargs();
        a.A = H; a.B = W; a.C = dB;
        a.M = J2; a.N = I2; a.K = I1 * J3; a.Ki = J3;
        a.sam = J3; a.sako = NN; a.saki = 1;
        a.sbn = J3; a.sbko = I2 * J3; a.sbki = 1;
        a.scm = I2; a.scn = 1;
        if ((rc = run_gemm<MATH>(a, 1, &sums, ws + p.off_P[1], st, "ttm_bwd_dB"))) return rc;
    }
    if (dC) {         // dC[j3][i3] = sum_{(i1,i2)} R[(i1,i2)][j3] X[(i1,i2)][i3]
        if (p.stream) {
            T *part = p.dc_splits > 1 ? reinterpret_cast<T *>(ws + p.off_P[2]) : static_cast<T *>(dC);
            const dim3 grid(unsigned(p.dc_splits), unsigned(ceil_div(I3, 64 * VE)));
            rc = launch("ttm_bwd_dC", st, [&] {
                auto go = [&](auto k) {
                    hipLaunchKernelGGL(k, grid, dim3(512), 0, st, Rt, Xt, part, M, int(I3), int(J3), p.dc_rows);
                };
                if (j3b == 1) go(k_bwd_dc<T, 1>);
                else if (j3b == 2) go(k_bwd_dc<T, 2>);
                else if (j3b == 3) go(k_bwd_dc<T, 3>);
                else go(k_bwd_dc<T, 4>);
            });
            if (p.dc_splits > 1) sums.add(part, dC, J3 * I3, p.dc_splits);
        } else {
            GemmArgs a = gargs();
            a.A = R; a.B = X; a.C = dC;
            a.M = J3; a.N = I3; a.K = M;
            a.sam = 1; a.saki = J3;
            a.sbn = 1; a.sbki = I3;
            a.scm = I3; a.scn = 1;
            rc = run_gemm<MATH>(a, 1, &sums, ws + p.off_P[2], st, "ttm_bwd_dC");
        }
        if (rc) return rc;
    }
    return sums.run(st);
}

int validate(const ttm_shape *s) {
    if (!s) return TTM_ERR_INVALID_ARG;
    for (int n = 0; n < 3; ++n)
        if (s->I[n] < 1 || s->J[n] < 1 || s->I[n] > (int64_t(1) << 31) || s->J[n] > (int64_t(1) << 31))
            return TTM_ERR_INVALID_ARG;
    if (checked_prod(checked_prod(s->I[0], s->I[1]), s->I[2]) < 0) return TTM_ERR_INVALID_ARG;
    if (checked_prod(checked_prod(s->J[0], s->J[1]), s->J[2]) < 0) return TTM_ERR_INVALID_ARG;
    return TTM_OK;
}

bool bwd_combo_ok(int dtype, int math) {
    return (dtype == TTM_F64 && math == TTM_MATH_F64) || (dtype == TTM_F32 && math == TTM_MATH_F32);
}

}  // namespace
}  // namespace ttm

using namespace ttm;

extern "C" {

size_t ttm_chain_backward_workspace_size(const ttm_shape *s, int dtype, int math) {
    if (validate(s) != TTM_OK || !bwd_combo_ok(dtype, math)) return 0;
    BwdPlan p;
    make_bwd_plan(*s, math, true, true, true, true, p);
    return std::max(p.total, p.f_total);
}

int ttm_chain_backward(const ttm_shape *s, const void *G, const void *X, const void *A, const void *B, const void *C,
                       int dtype, void *dX, void *dA, void *dB, void *dC, int math, void *ws, size_t ws_bytes,
                       void *stream) {
    int rc = validate(s);
    if (rc) return rc;
    if (!bwd_combo_ok(dtype, math)) return TTM_ERR_UNSUPPORTED;
    // every contraction length must fit the GEMM's 32-bit k index
    const int64_t k_max = std::max({s->I[0] * s->I[1], s->I[0] * s->J[2], s->J[1] * s->J[2], s->I[1], s->I[2], s->J[0]});
    if (k_max >= (int64_t(1) << 32)) return TTM_ERR_UNSUPPORTED;
    if (!G || !X || !A || !B || !C) return TTM_ERR_INVALID_ARG;
    if (!dX && !dA && !dB && !dC) return TTM_ERR_INVALID_ARG;
    const size_t e = dtype_size(dtype);
    const void *ins[5] = {G, X, A, B, C};
    void *outs[4] = {dX, dA, dB, dC};
    const size_t in_sz[5] = {size_t(s->J[0] * s->J[1] * s->J[2]) * e, size_t(s->I[0] * s->I[1] * s->I[2]) * e,
                             size_t(s->J[0] * s->I[0]) * e, size_t(s->J[1] * s->I[1]) * e, size_t(s->J[2] * s->I[2]) * e};
    const size_t out_sz[4] = {in_sz[1], in_sz[2], in_sz[3], in_sz[4]};
    for (int i = 0; i < 5; ++i)
        if (!aligned(ins[i], e)) return TTM_ERR_INVALID_ARG;
    for (int i = 0; i < 4; ++i)
        if (outs[i] && !aligned(outs[i], e)) return TTM_ERR_INVALID_ARG;
    // need only the workspace the requested gradients use; the size query reports the maximum
    BwdPlan p;
    make_bwd_plan(*s, math, dX != nullptr, dA != nullptr, dB != nullptr, dC != nullptr, p);
    // the fused kernels read X, C and write dX 16 bytes at a time
    const bool fused = p.fused && aligned(X, 16) && aligned(C, 16) && (!dX || aligned(dX, 16));
    if (fused) p.total = p.f_total;
    if (p.total > 0 && (!ws || ws_bytes < p.total)) return TTM_ERR_WORKSPACE;
    for (int i = 0; i < 4; ++i) {
        if (!outs[i]) continue;
        for (int j = 0; j < 5; ++j)
            if (overlaps(outs[i], out_sz[i], ins[j], in_sz[j])) return TTM_ERR_ALIAS;
        for (int j = i + 1; j < 4; ++j)
            if (outs[j] && overlaps(outs[i], out_sz[i], outs[j], out_sz[j])) return TTM_ERR_ALIAS;
        if (overlaps(outs[i], out_sz[i], ws, p.total)) return TTM_ERR_ALIAS;
    }
    for (int j = 0; j < 5; ++j)
        if (overlaps(ws, p.total, ins[j], in_sz[j])) return TTM_ERR_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char *w = static_cast<unsigned char *>(ws);
    if (fused) return run_fused(p, G, X, A, B, C, dX, dA, dB, dC, w, st);
    if (math == TTM_MATH_F64) return run_backward<M_F64>(p, G, X, A, B, C, dX, dA, dB, dC, w, st);
    return run_backward<M_F32>(p, G, X, A, B, C, dX, dA, dB, dC, w, st);
}

}  // extern "C"
