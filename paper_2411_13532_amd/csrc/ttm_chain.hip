// ttm_chain.hip -- Y = X x1 A x2 B x3 C on one MI355X (gfx950).
//
// Two to four kernels per call:
//   1. k_prep_factors : copy A, B, C into the workspace in the operand format
//      of the bf16 forms (hi/lo), with rows and columns zero-padded to the tile
//      grid so no later load needs a guard; in float and double only B and C,
//      only for the direct-to-LDS kernel, where their shapes need padding.
//   2. k_slab* : one workgroup per (i1, i2-range).  It streams its rows of X
//      once from HBM through an LDS double buffer and contracts mode 3 on the
//      matrix cores, W = X[i1, rows, :] C^T.  The W tile never reaches HBM: it
//      is the k-major operand of the mode-2 contraction V[i1] += B[:, rows] W,
//      from the registers it was summed in or through LDS.  At the end the
//      workgroup writes its partial V[i1] (J2 x J3, float) -- the only
//      intermediate that reaches HBM (1/I3 of X's element count times
//      J2*J3/I2, a few percent of X's bytes).
//   3. k_mode1_small : Y = A V_(1), summing the partials of V in a fixed order
//      (no atomics, so every call is bitwise reproducible); for a large V
//      k_mode1, and a fixed-order sum of its i1 splits where it has any.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>
#include <utility>

#include "ttm_device.hpp"
#include "ttm_host.hpp"

namespace ttm {

constexpr int SLAB_TM = 128;     // rows of X[i1] per tile
constexpr int SLAB_THREADS = 256;
constexpr int LC_TM = 256;       // the same of k_slab_lc

struct PrepArgs {
    const void *src[3];
    void *hi[3];
    void *lo[3];
    int64_t J[3], I[3], Jpad[3], ld[3];
    int perm32[3];   // 1: store columns in the mode-2 operand order (see below)
};

// Column position of source column c in a mode-2 bf16 operand row.  Inside
// every aligned block of 32 columns, accumulator rows 4g..4g+3 of the first
// 16-row block and 4g..4g+3 of the second one are the 8 k values of lane
// group g (slab_mode2); storing them next to each other lets one 16-byte
// load fetch the whole fragment.
__host__ __device__ inline int64_t mode2_col(int64_t c) {
    const int64_t q = c & 31, base = c - q;
    return q < 16 ? base + 8 * (q >> 2) + (q & 3) : base + 8 * ((q - 16) >> 2) + 4 + (q & 3);
}

// Factor n of shape J x I (row-major, float or double) -> padded Jpad x ld
// operand array(s).  For bfloat16 operands `hi` gets rne(v) and `lo` (when
// non-null) gets rne(v - hi).
template <typename ST, int MATH>
__global__ void __launch_bounds__(256) k_prep_factors(PrepArgs a) {
    const int f = blockIdx.y;
    const int64_t n = a.Jpad[f] * a.ld[f];
    const ST *src = static_cast<const ST *>(a.src[f]);
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x) {
        const int64_t r = e / a.ld[f], c = e % a.ld[f];
        const bool in = r < a.J[f] && c < a.I[f];
        if constexpr (MATH == M_BF16 || MATH == M_BF16X3) {
            const float v = in ? float(src[r * a.I[f] + c]) : 0.f;
            uint32_t h, l;
            bf16_split(v, h, l);
            const int64_t dst = a.perm32[f] ? r * a.ld[f] + mode2_col(c) : e;
            static_cast<uint16_t *>(a.hi[f])[dst] = uint16_t(h);
            if (a.lo[f]) static_cast<uint16_t *>(a.lo[f])[dst] = uint16_t(l);
        } else {
            typedef typename MathTraits<MATH>::fac_t FT;
            static_cast<FT *>(a.hi[f])[e] = in ? FT(src[r * a.I[f] + c]) : FT(0);
        }
    }
}

struct SlabArgs {
    const void *X;
    int64_t I1, I2, I3;
    const void *Chi, *Clo;  // [J3pad][ldc]
    int64_t ldc;
    const void *Bhi, *Blo;  // [J2pad][ldb]
    int64_t ldb;
    void *V;                // [I1][P][J2pad][J3pad]
    int64_t J2pad, J3pad;
    int P, S;
    int64_t rows_per_split;
    int64_t J2, J3;         // k_slab in float and double: B and C are the caller's (ldb = I2, ldc = I3)
};

// ---------------------------------------------------------------------------
// One 16-byte LDS operand group (VE values of the operand type LT) of X, of
// storage type XT.  load() takes any element-aligned address (gfx950 serves
// 16-byte loads at any alignment, so rows of odd length are read as wide as
// aligned ones); load_some() reads the first n values only; shift() (float and
// double factors) moves a group that would end past the tensor, and was loaded
// d values before its place, into place; keep() zeroes what lies past the
// row's end or the row range.  shift() and keep() run just before store(), not
// after the load: the registers are touched only once the group is needed.
// ---------------------------------------------------------------------------
typedef u32x4 u32x4_u __attribute__((aligned(2)));
typedef u32x2 u32x2_u __attribute__((aligned(2)));

template <typename T, int VE> __device__ __forceinline__ void shift_values(T (&v)[VE], int d) {
#pragma unroll
    for (int s = 1; s < VE; s *= 2)
#pragma unroll
        for (int e = 0; e < VE; ++e) v[e] = d & s ? (e + s < VE ? v[e + s < VE ? e + s : 0] : T(0)) : v[e];
}

template <typename XT, typename LT> struct XGroup;

template <typename T> struct XGroup<T, T> {          // same type: one 16-byte load
    static constexpr int VE = 16 / sizeof(T), REGS = 4;
    V16 raw;
    __device__ void clear() { raw = zero16(); }
    __device__ void load(const T *p) { raw.u = *reinterpret_cast<const u32x4_u *>(p); }
    __device__ void load_some(const T *p, int n) {
        T tmp[VE];
#pragma unroll
        for (int e = 0; e < VE; ++e) tmp[e] = e < n ? p[e] : T(0);
        __builtin_memcpy(&raw, tmp, 16);
    }
    __device__ void shift(int d) {
        T tmp[VE];
        __builtin_memcpy(tmp, &raw, 16);
        shift_values(tmp, d);
        __builtin_memcpy(&raw, tmp, 16);
    }
    __device__ void keep(int n) {
        T tmp[VE];
        __builtin_memcpy(tmp, &raw, 16);
#pragma unroll
        for (int e = 0; e < VE; ++e) tmp[e] = e < n ? tmp[e] : T(0);
        __builtin_memcpy(&raw, tmp, 16);
    }
    __device__ void store(unsigned char *hi, unsigned char *) const { *reinterpret_cast<u32x4 *>(hi) = raw.u; }
};

template <> struct XGroup<uint16_t, float> {        // bf16 X, float operands: 8-byte load
    static constexpr int VE = 4, REGS = 2;
    u32x2 raw;
    __device__ void clear() { raw = u32x2{0u, 0u}; }
    __device__ void load(const uint16_t *p) { raw = *reinterpret_cast<const u32x2_u *>(p); }
    __device__ void load_some(const uint16_t *p, int n) {
        uint32_t h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = e < n ? p[e] : 0u;
        raw = u32x2{pack2(h[0], h[1]), pack2(h[2], h[3])};
    }
    __device__ void keep(int n) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t m = n > 2 * e + 1 ? ~0u : (n > 2 * e ? 0xffffu : 0u);
            raw[e] &= m;
        }
    }
    __device__ void store(unsigned char *hi, unsigned char *) const {
        f32x4 v;
        v[0] = __uint_as_float(raw[0] << 16);
        v[1] = __uint_as_float(raw[0] & 0xffff0000u);
        v[2] = __uint_as_float(raw[1] << 16);
        v[3] = __uint_as_float(raw[1] & 0xffff0000u);
        *reinterpret_cast<f32x4 *>(hi) = v;
    }
};

template <> struct XGroup<float, uint16_t> {        // float X, bf16 operands: 32-byte load, split on store
    static constexpr int VE = 8, REGS = 8;
    V16 raw0, raw1;
    __device__ void clear() { raw0 = raw1 = zero16(); }
    __device__ void load(const float *p) {
        raw0.u = *reinterpret_cast<const u32x4_u *>(p);
        raw1.u = *reinterpret_cast<const u32x4_u *>(p + 4);
    }
    __device__ void load_some(const float *p, int n) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            raw0.f[e] = e < n ? p[e] : 0.f;
            raw1.f[e] = e + 4 < n ? p[e + 4] : 0.f;
        }
    }
    __device__ void keep(int n) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            raw0.f[e] = e < n ? raw0.f[e] : 0.f;
            raw1.f[e] = e + 4 < n ? raw1.f[e] : 0.f;
        }
    }
    __device__ void store(unsigned char *hi, unsigned char *lo) const {
        const float v[8] = {raw0.f[0], raw0.f[1], raw0.f[2], raw0.f[3], raw1.f[0], raw1.f[1], raw1.f[2], raw1.f[3]};
        u32x4 h, l;
        bf16_split8(v, h, lo ? &l : nullptr);
        *reinterpret_cast<u32x4 *>(hi) = h;
        if (lo) *reinterpret_cast<u32x4 *>(lo) = l;
    }
};

// Tile of the register-staged kernel: 64 * MB rows of X[i1] by CB blocks of
// 16 columns j3, in chunks of 128 bytes of operand per row (rows padded to 144
// in LDS: 16 rows then start in 16 different 16-byte bank groups).  The X and
// C chunks take two LDS slots; the W tile that hands the rows over to the
// mode-2 step takes the slot just consumed where it fits, LDS of its own
// elsewhere.  WR: partials of V per row split.  Plain bf16 rounds the sum of
// the partials to bf16 before mode 1, so a sum taken in another order moves
// some values by a bf16 rounding: there the partials, their splits and the
// order of the rows in them are those of the direct-to-LDS kernels' waves.
struct SlabTile {
    int MB, TM, WR, xb, cb, slot, wrow, wb, walias, lds;
};
constexpr int SLAB_ROWB = 144;
constexpr SlabTile slab_tile(int math, bool x_float, int CB) {
    SlabTile t = {};
    const bool x3 = math == M_BF16X3, xlo = x3 && x_float;
    const int lt = math == M_F64 ? 8 : math == M_F32 ? 4 : 2;
    // 128 rows (each C fragment read from LDS feeds twice the products) where
    // two workgroups still fit a compute unit, in LDS and in registers
    t.MB = (math == M_BF16 && CB <= (x_float ? 4 : 6)) || (x3 && !xlo && CB <= 4) ? 2 : 1;
    t.TM = 64 * t.MB;
    t.WR = math == M_BF16 && CB <= 2 ? 4 / CB : 1;
    t.xb = t.TM * SLAB_ROWB;
    t.cb = CB * 16 * SLAB_ROWB;
    t.slot = t.xb * (xlo ? 2 : 1) + t.cb * (x3 ? 2 : 1);
    t.wrow = t.TM * lt + 16;
    t.wb = CB * 16 * t.wrow;
    t.walias = t.wb * (x3 ? 2 : 1) <= t.slot;
    t.lds = 2 * t.slot + (t.walias ? 0 : t.wb * (x3 ? 2 : 1));
    return t;
}
// Resident waves per SIMD the kernel's registers are cut for: as many as its
// tile has room for (without the bound the allocator gave up a wave for a few
// values more: 512^3 -> 64 in float 126 registers, or 145).
constexpr int slab_waves(int math, bool x_float, int CB, int JB) {
    if (JB == 8 || math == M_BF16X3) return math == M_F32 && CB <= 4 ? 3 : 2;
    if (math == M_F32) return CB == 1 ? 5 : CB <= 4 || (!x_float && JB == 1) ? 4 : 3;
    if (math == M_F64) return CB <= 2 || JB <= 2 ? 3 : 2;
    if (!x_float && CB == 2 && JB <= 2) return 4;
    return CB <= 2 || CB == 8 || (x_float ? CB == 6 || (CB == 3 && JB == 1) : CB <= 4) ? 3 : 2;
}
// A group loaded from `off`, or from the tensor's last whole group where it
// would end past it, with its first n values in place and zeros after them.
// (A tensor shorter than a group was not loaded at all: value by value here.)
template <typename G, typename T>
__device__ __forceinline__ void place_group(G &x, const T *base, int64_t off, int64_t total, int n) {
    if (total < G::VE) {
        const int64_t m = total - off;
        x.load_some(base + (m > 0 ? off : 0), int(m < n ? m : n));
        wait_vmcnt<0>();   // here, so that the common path need not wait for these
    } else {
        const int64_t d = off - (total - G::VE);
        x.shift(d > 0 ? int(d) : 0);
        x.keep(n);
    }
}

template <int MATH, typename XT, int CB> struct SlabCfg {
    typedef MathTraits<MATH> TR;
    typedef typename TR::lds_t LT;
    static constexpr int VE = TR::VE;
    static constexpr int KG = TR::KG;             // k per k-group (64 bytes of LT per row)
    static constexpr int KC = 2 * KG;             // k per chunk
    static constexpr bool X3 = MATH == M_BF16X3;
    static constexpr bool XLO = X3 && std::is_same<XT, float>::value;
    static constexpr SlabTile T = slab_tile(MATH, std::is_same<XT, float>::value, CB);
    static constexpr int MB = T.MB, TM = T.TM, WR = T.WR, ROWB = SLAB_ROWB, XB = T.xb, CBY = T.cb, SLOT = T.slot;
    static constexpr int WROW = T.wrow, WB = T.wb, LDS = T.lds;
    static constexpr bool WALIAS = T.walias != 0;
    static constexpr int XG = TM * 8 / SLAB_THREADS;               // 16-byte X groups per thread and chunk
    static constexpr int CG = (CB * 128 + SLAB_THREADS - 1) / SLAB_THREADS;   // the same for C
};

// Mode-2 step: V[jb][nb] += B[j2 rows, tile rows] * W[tile rows, cols].
// f32/f64: per 16-row block, the accumulator register r of lane (g, c) is
// W[acc_row(g, r)][c], so MFMA r takes k-slot g <-> row acc_row(g, r).
template <int MATH, int MB, int NBW, int JB>
__device__ __forceinline__ void slab_mode2(typename MathTraits<MATH>::accv_t (&vacc)[JB][NBW],
                                           const typename MathTraits<MATH>::accv_t (&wacc)[MB][NBW],
                                           const SlabArgs &a, int jbase, int64_t wrow0, int l16, int g) {
    if constexpr (MATH == M_F32 || MATH == M_F64) {
        typedef typename MathTraits<MATH>::fac_t FT;
        const FT *Bp = static_cast<const FT *>(a.Bhi);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                {
                    const FT *brow = Bp + int64_t((jbase + jb) * 16 + l16) * a.ldb + wrow0 + mb * 16;
                    FT bv[4];
                    if constexpr (MATH == M_F32) {
                        V16 t = ld16(brow + 4 * g);        // rows 4g .. 4g+3
#pragma unroll
                        for (int r = 0; r < 4; ++r) bv[r] = t.f[r];
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) bv[r] = brow[MathTraits<MATH>::acc_row(g, r)];
                    }
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            if constexpr (MATH == M_F32) vacc[jb][nb] = mfma_f32(bv[r], wacc[mb][nb][r], vacc[jb][nb]);
                            else vacc[jb][nb] = mfma_f64(bv[r], wacc[mb][nb][r], vacc[jb][nb]);
                        }
                }
            }
            // keep the next block's loads from being hoisted (register pressure)
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        // bf16: two stacked 16-row blocks give a lane the 8 values
        // {W[32p + 4g + e], W[32p + 16 + 4g + e]}, e = 0..3 -> one k-slot group;
        // the B operand stores those 8 columns contiguously (mode2_col).
        const uint16_t *Bh = static_cast<const uint16_t *>(a.Bhi);
        const uint16_t *Bl = static_cast<const uint16_t *>(a.Blo);
#pragma unroll
        for (int p = 0; p < MB / 2; ++p) {
            u32x4 wh[NBW], wl[NBW];
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                const float v[8] = {wacc[2 * p][nb][0], wacc[2 * p][nb][1], wacc[2 * p][nb][2], wacc[2 * p][nb][3],
                                    wacc[2 * p + 1][nb][0], wacc[2 * p + 1][nb][1], wacc[2 * p + 1][nb][2],
                                    wacc[2 * p + 1][nb][3]};
                if constexpr (MATH == M_BF16X3) bf16_split8(v, wh[nb], &wl[nb]);
                else wh[nb] = bf16_round8(v);
            }
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                const int64_t off = int64_t((jbase + jb) * 16 + l16) * a.ldb + wrow0 + 32 * p + 8 * g;
                const u32x4 bh = ld16(Bh + off).u;
                if constexpr (MATH == M_BF16X3) {
                    const u32x4 bl = ld16(Bl + off).u;
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) {
                        vacc[jb][nb] = mfma_bf16(bh, wh[nb], vacc[jb][nb]);
                        vacc[jb][nb] = mfma_bf16(bh, wl[nb], vacc[jb][nb]);
                        vacc[jb][nb] = mfma_bf16(bl, wh[nb], vacc[jb][nb]);
                    }
                } else {
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) vacc[jb][nb] = mfma_bf16(bh, wh[nb], vacc[jb][nb]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// k_slab: X through registers into LDS, for any row length, alignment and
// storage type of X.  Four waves, each owning 16 * MB rows of the tile and all
// of its columns, so that J3 is padded to 16 and not to four waves' columns,
// waves whose rows lie past I2 do no products, and X and C are each read from
// LDS once per 16 rows.  The chunk loop keeps X two chunks ahead in registers
// and C one (issued before X: vector-memory loads complete in order, so a wait
// for a factor issued after an X fetch would wait for its HBM trip too).
// The mode-2 step V[i1] += B[:, rows] W takes W through LDS, so that its
// (j2, j3) blocks are dealt to the waves: V is held once per workgroup, not
// once per wave, and one partial per row split reaches HBM.
// Bound by HBM in the bf16 forms, by the matrix cores in float and double on
// full chips, by latency (a chunk's barrier, a fetch's trip) on small ones.
// Measured, whole chains: 385 x 510 x 771 -> 48 x 50 x 70 in bf16, odd rows
// read value by value with the waits of one chunk exposed: 287 us, now 113 us;
// 181 x 210 x 155 -> 24 x 30 x 41 in double 59 us, now 39.5 us;
// 332 x 409 x 232 -> 65 x 80 x 48 in double 567 us, now 205 us.  With one column
// block in plain bf16 and many short workgroups (i1 in the hundreds) the kernel
// that handed W over in registers, at four and five workgroups a compute unit
// where three fit now, was ahead: 888 x 16 x 64 -> 64 x 8 x 8 17.3 us, now 21.3.
template <int MATH, typename XT, int CB, int JB>
__global__ void __launch_bounds__(SLAB_THREADS, slab_waves(MATH, std::is_same<XT, float>::value, CB, JB)) k_slab(const SlabArgs a) {
    typedef SlabCfg<MATH, XT, CB> CF;
    typedef typename CF::TR TR;
    typedef typename CF::LT LT;
    typedef typename TR::accv_t accv_t;
    typedef typename TR::acc_t acc_t;
    typedef typename TR::fac_t FT;
    constexpr int MB = CF::MB, TM = CF::TM, KG = CF::KG, KC = CF::KC, VE = CF::VE, XG = CF::XG, CG = CF::CG;
    constexpr bool X3 = CF::X3, XLO = CF::XLO;
    constexpr int NJ = JB > 4 ? JB / 4 : 1;                    // j2 blocks of a wave's share of V
    constexpr int NC = JB >= 4 ? CB : JB == 2 ? (CB + 1) / 2 : (CB + 3) / 4;   // its j3 blocks
    constexpr int KQ = TM / KG;                                // k-groups of a mode-2 step
    constexpr int WR = CF::WR;                                 // partials of V, KQ / WR k-groups of each tile
    constexpr bool RAGGED = NC * (JB >= 4 ? 1 : 4 / JB) != CB;  // some waves' shares end past the last j3 block
    static_assert(JB == 1 || JB == 2 || JB == 4 || JB == 8, "j2 blocks");

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;

    const int64_t i1 = blockIdx.x / a.S;
    const int s = int(blockIdx.x % a.S);
    const int64_t row_begin = int64_t(s) * a.rows_per_split;
    const int64_t row_end = a.I2 < row_begin + a.rows_per_split ? a.I2 : row_begin + a.rows_per_split;
    const int64_t nrows = row_end > row_begin ? row_end - row_begin : 0;
    const int64_t col0 = int64_t(blockIdx.y) * (CB * 16);
    // first j2 and j3 block of this wave's share
    const int jb0 = int(blockIdx.z) * JB + (JB >= 4 ? wave * NJ : JB == 2 ? (wave & 1) : 0);
    const int nb0 = JB >= 4 ? 0 : JB == 2 ? (wave >> 1) * NC : wave * NC;

    const XT *Xs = static_cast<const XT *>(a.X) + i1 * a.I2 * a.I3;
    // values of X from this slab's start on, and where its last whole group
    // starts (an X shorter than a group is only read value by value: there the
    // wide loads, whose values are not used, go to V)
    const int64_t left = (a.I1 - i1) * a.I2 * a.I3;
    const bool tiny = a.I1 * a.I2 * a.I3 < VE;
    const int64_t wide = tiny ? 0 : left - VE;
    const XT *Xl = tiny ? static_cast<const XT *>(a.V) : Xs;
    const int nk = int(ceil_div(a.I3, KC)), ntiles = int(ceil_div(nrows, TM));
    const int64_t nq = int64_t(ntiles) * nk;
    const FT *Ch = static_cast<const FT *>(a.Chi), *Cl = static_cast<const FT *>(a.Clo);
    const FT *Bh = static_cast<const FT *>(a.Bhi), *Bl = static_cast<const FT *>(a.Blo);

    auto xslot = [&](int slot, int lo) -> unsigned char * { return smem + slot * CF::SLOT + lo * CF::XB; };
    auto cslot = [&](int slot, int lo) -> unsigned char * {
        return smem + slot * CF::SLOT + (XLO ? 2 : 1) * CF::XB + lo * CF::CBY;
    };

    XGroup<XT, LT> px[2][XG];
    V16 pch[CG], pcl[CG];                                      // (bf16 forms)
    const int gr = tid >> 3, gp = tid & 7;                     // row and 16-byte piece of a thread's first group
    // Offsets of a thread's rows of the tile being fetched (rows past the range
    // read its last one), formed once per tile: a chunk's addresses then take
    // two 64-bit additions each.
    int64_t rowoff[XG];
    bool near_end = false;             // some group of the tile may end past X
    auto set_rows = [&](int64_t t) __attribute__((always_inline)) {
        const int64_t r0 = row_begin + t * TM;
        const int64_t last = (r0 + TM < row_end ? r0 + TM : row_end) - 1;
        near_end = (last + 1) * a.I3 > wide;
#pragma unroll
        for (int j = 0; j < XG; ++j) {
            const int64_t row = r0 + gr + 32 * j;
            rowoff[j] = (row < last ? row : last) * a.I3;
        }
    };
    auto fetch_x = [&](int kc, XGroup<XT, LT> (&x)[XG]) __attribute__((always_inline)) {
        const int64_t k = int64_t(kc) * KC + gp * VE, kk = k < a.I3 ? k : 0;
        int64_t off[XG];
#pragma unroll
        for (int j = 0; j < XG; ++j) off[j] = rowoff[j] + kk;
        if (near_end) {
#pragma unroll
            for (int j = 0; j < XG; ++j) off[j] = off[j] < wide ? off[j] : wide;
        }
#pragma unroll
        for (int j = 0; j < XG; ++j) x[j].load(Xl + off[j]);
    };
    auto store_x = [&](int slot, int64_t t, int64_t kc, XGroup<XT, LT> (&x)[XG]) __attribute__((always_inline)) {
        const int64_t r0 = row_begin + t * TM;
        const int64_t end = r0 + TM < row_end ? r0 + TM : row_end;
        if (end * a.I3 > wide && int64_t(kc + 1) * KC > a.I3) {
            // X's last values: a group that would end past them was fetched
            // from before its place, and is read again value by value
#pragma unroll
            for (int j = 0; j < XG; ++j) {
                const int64_t row = r0 + gr + 32 * j, k = int64_t(kc) * KC + gp * VE, off = row * a.I3 + k;
                if (row < end && k < a.I3 && off + VE > left) x[j].load_some(Xs + off, int(left - off));
            }
            wait_vmcnt<0>();   // here, so that the common path need not wait for these
        }
        if (r0 + TM > row_end || int64_t(kc + 1) * KC > a.I3) {       // rows or k past the end: zeros
            const int64_t kleft = a.I3 - (int64_t(kc) * KC + gp * VE);
            const int n = kleft >= VE ? VE : (kleft > 0 ? int(kleft) : 0);
#pragma unroll
            for (int j = 0; j < XG; ++j) x[j].keep(r0 + gr + 32 * j < row_end ? n : 0);
        }
#pragma unroll
        for (int j = 0; j < XG; ++j) {
            const int off = (gr + 32 * j) * CF::ROWB + gp * 16;
            x[j].store(xslot(slot, 0) + off, XLO ? xslot(slot, 1) + off : nullptr);
        }
    };
    // (the last half of an odd number of column blocks: waves 0 and 1 only)
    auto c_in = [&](int u) { return CB % 2 == 0 || u + 1 < CG || wave < 2; };
    // C: in the bf16 forms the padded operand array, in float and double the
    // caller's factor (rows past J3 repeat the last one: their columns of V are
    // not read)
    constexpr bool RAW = MATH == M_F32 || MATH == M_F64;
    typedef XGroup<FT, FT> FG;
    FG pc[CG];
    const int64_t ctotal = a.J3 * a.I3, cwide = ctotal < VE ? 0 : ctotal - VE;
    const FT *Cs = RAW && ctotal < VE ? static_cast<const FT *>(a.V) : Ch;
    int64_t coff[CG];
#pragma unroll
    for (int u = 0; u < CG; ++u) {
        const int64_t row = col0 + gr + 32 * u;
        if constexpr (RAW) coff[u] = (row < a.J3 ? row : a.J3 - 1) * a.I3;
        else coff[u] = row * a.ldc + gp * VE;
    }
    auto fetch_c = [&](int kc) __attribute__((always_inline)) {
        if constexpr (RAW) {
            const int64_t k = int64_t(kc) * KC + gp * VE, kk = k < a.I3 ? k : 0;
#pragma unroll
            for (int u = 0; u < CG; ++u)
                if (c_in(u)) {
                    const int64_t off = coff[u] + kk;
                    pc[u].load(Cs + (off < cwide ? off : cwide));
                }
        } else {
            const FT *ch = Ch + int64_t(kc) * KC, *cl = Cl + int64_t(kc) * KC;
#pragma unroll
            for (int u = 0; u < CG; ++u)
                if (c_in(u)) {
                    pch[u] = ld16(ch + coff[u]);
                    if constexpr (X3) pcl[u] = ld16(cl + coff[u]);
                }
        }
    };
    auto store_c = [&](int slot, int kc) __attribute__((always_inline)) {
        if constexpr (RAW) {
            if ((int64_t(kc) + 1) * KC > a.I3) {
                const int64_t k = int64_t(kc) * KC + gp * VE, kleft = a.I3 - k;
                const int n = kleft >= VE ? VE : (kleft > 0 ? int(kleft) : 0);
#pragma unroll
                for (int u = 0; u < CG; ++u)
                    if (c_in(u)) place_group(pc[u], Ch, coff[u] + (n > 0 ? k : 0), ctotal, n);
            }
        }
#pragma unroll
        for (int u = 0; u < CG; ++u)
            if (c_in(u)) {
                const int off = (gr + 32 * u) * CF::ROWB + gp * 16;
                if constexpr (RAW) {
                    *reinterpret_cast<u32x4 *>(cslot(slot, 0) + off) = pc[u].raw.u;
                } else {
                    *reinterpret_cast<u32x4 *>(cslot(slot, 0) + off) = pch[u].u;
                    if constexpr (X3) *reinterpret_cast<u32x4 *>(cslot(slot, 1) + off) = pcl[u].u;
                }
            }
    };

    accv_t vacc[WR][NJ][NC], wacc[MB][CB];
#pragma unroll
    for (int w = 0; w < WR; ++w)
#pragma unroll
        for (int i = 0; i < NJ; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j) vacc[w][i][j] = zero_accv<accv_t>();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < CB; ++nb) wacc[mb][nb] = zero_accv<accv_t>();

    // B's fragments of a tile's mode-2 step (float and double: from the
    // caller's factor, rows past J2 repeating the last one)
    FG fbh[NJ][KQ], fbl[NJ][KQ];
    const int64_t btotal = a.J2 * a.I2, bwide = btotal < VE ? 0 : btotal - VE;
    const FT *Bs = RAW && btotal < VE ? static_cast<const FT *>(a.V) : Bh;
    int64_t boff[NJ];
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        const int64_t row = int64_t(jb0 + i) * 16 + l16;
        boff[i] = RAW ? (row < a.J2 ? row : a.J2 - 1) * a.I2 : row * a.ldb;
    }
    auto fetch_b = [&](int64_t t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NJ; ++i)
#pragma unroll
            for (int kq = 0; kq < KQ; ++kq) {
                const int64_t k = row_begin + t * TM + kq * KG + g * VE;
                if constexpr (RAW) {
                    const int64_t off = boff[i] + (k < a.I2 ? k : 0);
                    fbh[i][kq].load(Bs + (off < bwide ? off : bwide));
                } else {
                    fbh[i][kq].raw = ld16(Bh + boff[i] + k);
                    if constexpr (X3) fbl[i][kq].raw = ld16(Bl + boff[i] + k);
                }
            }
    };
    auto place_b = [&](int64_t t) __attribute__((always_inline)) {
        if constexpr (RAW) {
            if (row_begin + (t + 1) * TM <= a.I2) return;
#pragma unroll
            for (int i = 0; i < NJ; ++i)
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    const int64_t k = row_begin + t * TM + kq * KG + g * VE, kleft = a.I2 - k;
                    const int n = kleft >= VE ? VE : (kleft > 0 ? int(kleft) : 0);
                    place_group(fbh[i][kq], Bh, boff[i] + (n > 0 ? k : 0), btotal, n);
                }
        }
    };
    auto mode2 = [&](int64_t t, int slot) __attribute__((always_inline)) {
        // rows past the range, in the wave that the range ends in: X's zeros
        // times an infinite entry of C are NaN, which B's zeros would pass on
        // to every j2 (later waves have formed no products; in bf16 below, as
        // the values are packed; a split infinity is NaN by itself)
        const int live = int(row_end - row_begin - t * TM) - wave * (16 * MB);
        if (RAW && live > 0 && live < 16 * MB) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool in = mb * 16 + TR::acc_row(g, r) < live;
#pragma unroll
                    for (int nb = 0; nb < CB; ++nb) wacc[mb][nb][r] = in ? wacc[mb][nb][r] : acc_t(0);
                }
        }
        unsigned char *wh = smem + (CF::WALIAS ? slot * CF::SLOT : 2 * CF::SLOT), *wl = wh + CF::WB;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < CB; ++nb) {
                const int row = (wave * MB + mb) * 16, off = (nb * 16 + l16) * CF::WROW;
                const accv_t w = wacc[mb][nb];
                if constexpr (MATH == M_F32) {
                    *reinterpret_cast<f32x4 *>(wh + off + (row + 4 * g) * 4) = w;
                } else if constexpr (MATH == M_F64) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) *reinterpret_cast<double *>(wh + off + (row + TR::acc_row(g, r)) * 8) = w[r];
                } else {
                    // the operand order of B's columns (mode2_col)
                    const int pos = ((row & ~31) + 8 * g + ((row >> 4) & 1) * 4) * 2;
                    uint32_t h0, h1, l0, l1;
                    if constexpr (X3) {
                        bf16_split2(w[0], w[1], h0, l0);
                        bf16_split2(w[2], w[3], h1, l1);
                        *reinterpret_cast<u32x2 *>(wl + off + pos) = u32x2{l0, l1};
                    } else {
                        const int n = live - mb * 16 - 4 * g;
                        h0 = cvt_pk_bf16(w[0], w[1]) & (n >= 2 ? ~0u : n == 1 ? 0xffffu : 0u);
                        h1 = cvt_pk_bf16(w[2], w[3]) & (n >= 4 ? ~0u : n == 3 ? 0xffffu : 0u);
                    }
                    *reinterpret_cast<u32x2 *>(wh + off + pos) = u32x2{h0, h1};
                }
                wacc[mb][nb] = zero_accv<accv_t>();
            }
        __syncthreads();
#pragma unroll
        for (int kq = 0; kq < KQ; ++kq)
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int nb = RAGGED && nb0 + j >= CB ? CB - 1 : nb0 + j;   // past the end: not stored
                const int off = (nb * 16 + l16) * CF::WROW + kq * 64 + g * 16;
                const V16 w = {*reinterpret_cast<const u32x4 *>(wh + off)};
                V16 wlo;
                if constexpr (X3) wlo.u = *reinterpret_cast<const u32x4 *>(wl + off);
#pragma unroll
                for (int i = 0; i < NJ; ++i) {
                    mma_kgroup<X3 ? M_BF16 : MATH>(vacc[kq / (KQ / WR)][i][j], fbh[i][kq].raw, w);
                    if constexpr (X3) {
                        mma_kgroup<M_BF16>(vacc[kq / (KQ / WR)][i][j], fbh[i][kq].raw, wlo);
                        mma_kgroup<M_BF16>(vacc[kq / (KQ / WR)][i][j], fbl[i][kq].raw, w);
                    }
                }
            }
        if constexpr (CF::WALIAS) __syncthreads();             // the slot is filled again by the next chunk
    };

    int t = 0, kc = 0, t1 = 0, kc1 = 0, t2, kc2;
    auto products = [&](auto SLOT) __attribute__((always_inline)) {
        constexpr int S = decltype(SLOT)::value;
        if (row_begin + t * TM + wave * (16 * MB) < row_end) {
#pragma unroll
            for (int kg = 0; kg < 2; ++kg) {
                V16 ah[MB], al[MB];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int off = ((wave * MB + mb) * 16 + l16) * CF::ROWB + kg * 64 + g * 16;
                    ah[mb].u = *reinterpret_cast<const u32x4 *>(xslot(S, 0) + off);
                    if constexpr (XLO) al[mb].u = *reinterpret_cast<const u32x4 *>(xslot(S, 1) + off);
                }
#pragma unroll
                for (int nb = 0; nb < CB; ++nb) {
                    const int off = (nb * 16 + l16) * CF::ROWB + kg * 64 + g * 16;
                    V16 ch, cl;
                    ch.u = *reinterpret_cast<const u32x4 *>(cslot(S, 0) + off);
                    if constexpr (X3) cl.u = *reinterpret_cast<const u32x4 *>(cslot(S, 1) + off);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) {
                        mma_kgroup<X3 ? M_BF16 : MATH>(wacc[mb][nb], ah[mb], ch);
                        if constexpr (X3) mma_kgroup<M_BF16>(wacc[mb][nb], ah[mb], cl);
                        if constexpr (XLO) mma_kgroup<M_BF16>(wacc[mb][nb], al[mb], ch);
                    }
                }
            }
        }
    };
    // chunks q, q + 1 and q + 2 (past the last one the last again: the fetches
    // have no condition, so that the number of loads in flight, which the waits
    // count, is the same on every path; for the same reason every step stores
    // the next chunk and the steps come in pairs)
    auto next = [&](int &tt, int &kk) {
        if (kk + 1 < nk) { ++kk; return false; }
        if (tt + 1 == ntiles) return false;
        kk = 0;
        ++tt;
        return true;
    };
    // One chunk in all, in the bf16 forms with one column block, where tensors
    // of few columns have many such workgroups: nothing is fetched ahead (928 x
    // 48 x 48 -> 7, 6, 7 in bf16 20.3 us with the chunk fetched three times, so
    // 18.6).
    constexpr bool SINGLE = !RAW && CB == 1;
    if (SINGLE && nq == 1) {
        fetch_c(0);
        fetch_b(0);
        set_rows(0);
        fetch_x(0, px[0]);
        store_c(0, 0);
        store_x(0, 0, 0, px[0]);
        __syncthreads();
        products(std::integral_constant<int, 0>{});
        __syncthreads();
        mode2(0, 0);
    } else {
        fetch_c(0);
        set_rows(0);
        fetch_x(0, px[0]);
        if (next(t1, kc1)) set_rows(t1);
        fetch_x(kc1, px[1]);
        t2 = t1; kc2 = kc1;
        if (next(t2, kc2)) set_rows(t2);
        store_c(0, 0);
        store_x(0, 0, 0, px[0]);
        __syncthreads();
        auto step = [&](auto SLOT) __attribute__((always_inline)) {
            constexpr int S = decltype(SLOT)::value;
            fetch_c(kc1);
            if (kc == nk - 1) fetch_b(t);
            fetch_x(kc2, px[S]);
            __builtin_amdgcn_sched_barrier(0);
            products(SLOT);
            store_c(1 - S, kc1);                // (after the last chunk: that chunk again, which nothing reads)
            store_x(1 - S, t1, kc1, px[1 - S]);
            __syncthreads();
            if (kc == nk - 1) {
                place_b(t);
                mode2(t, S);
            }
            t = t1; kc = kc1;
            t1 = t2; kc1 = kc2;
            if (next(t2, kc2)) set_rows(t2);
        };
        for (int64_t q = nq; q >= 2; q -= 2) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
        }
        if (nq & 1) step(std::integral_constant<int, 0>{});
    }

    // V[i1][s * WR + w][j2][j3]: lane (g, c) register r of a block holds row acc_row(g, r), column c
    acc_t *Vp = static_cast<acc_t *>(a.V) + (i1 * a.P + s * WR) * a.J2pad * a.J3pad;
#pragma unroll
    for (int w = 0; w < WR; ++w)
#pragma unroll
        for (int i = 0; i < NJ; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                if (RAGGED && nb0 + j >= CB) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t j2 = int64_t(jb0 + i) * 16 + TR::acc_row(g, r);
                    Vp[(w * a.J2pad + j2) * a.J3pad + col0 + (nb0 + j) * 16 + l16] = vacc[w][i][j][r];
                }
            }
}

// ---------------------------------------------------------------------------
// k_slab_rows: the same computation as k_slab for at most 16 columns j3 and
// short walks, where a workgroup's time is not its bytes: four waves of 32 rows
// each, X one chunk ahead through one register set, W handed to the mode-2 step
// in the registers it was summed in (no W tile, no barriers for it), four
// workgroups a compute unit.  Rows past I2 are not fetched.  Float and double:
// all of C in LDS from the start, B read where it is, the waves' shares of V
// added at the end.  Plain bf16: C's fragments from L2, a partial of V per wave,
// as in k_slab and to the same bits.  Bound by the latency of the chunks' trips
// and by the number of workgroups that share them.  The whole chain, k_slab and
// this one: 769 x 10 x 269 -> 1, 5, 2 in bf16 29.9 and 18.4 us; 941 x 928 x 16 ->
// 1, 3, 1 in float 54.5 and 29.2; 808 x 635 x 6 -> 35, 8, 2 in double 70 and 35;
// 424 x 392 x 48 -> 8, 15, 16 in double 39.9 and 24.9.
// ---------------------------------------------------------------------------
constexpr int slab_rows_lds(int64_t nk) { return (2 * SLAB_TM + 16 * int(nk)) * SLAB_ROWB; }   // X twice, all of C (float and double)
template <int MATH, typename XT, int JB>
__global__ void __launch_bounds__(SLAB_THREADS, JB == 8 ? 3 : 4) k_slab_rows(const SlabArgs a) {
    typedef MathTraits<MATH> TR;
    typedef typename TR::lds_t LT;
    typedef typename TR::fac_t FT;
    typedef typename TR::acc_t acc_t;
    typedef typename TR::accv_t accv;
    constexpr bool RAW = MATH != M_BF16;
    constexpr int VE = TR::VE, KG = TR::KG, KC = 2 * KG, GROUPS = SLAB_TM * 8 / SLAB_THREADS, TILE = SLAB_TM * SLAB_ROWB;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t i1 = blockIdx.x / a.S;
    const int s = int(blockIdx.x % a.S);
    const int64_t row_begin = int64_t(s) * a.rows_per_split;
    const int64_t row_end = a.I2 < row_begin + a.rows_per_split ? a.I2 : row_begin + a.rows_per_split;
    const int jbase = int(blockIdx.z) * JB;
    const XT *Xs = static_cast<const XT *>(a.X) + i1 * a.I2 * a.I3;
    const FT *Ch = static_cast<const FT *>(a.Chi), *Bh = static_cast<const FT *>(a.Bhi);
    const int nk = int(ceil_div(a.I3, KC)), ntiles = int(ceil_div(row_end - row_begin, SLAB_TM));
    accv vacc[JB][1], wacc[2][1];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) vacc[jb][0] = zero_accv<accv>();
    XGroup<XT, LT> x[GROUPS];
    const int gr = tid >> 3, gp = tid & 7;             // row and 16-byte piece of a thread's first group
    auto fetch = [&](int t, int kc) __attribute__((always_inline)) {
        const int64_t k = int64_t(kc) * KC + gp * VE, kleft = a.I3 - k;
#pragma unroll
        for (int j = 0; j < GROUPS; ++j) {
            const int64_t row = row_begin + int64_t(t) * SLAB_TM + gr + 32 * j;
            const XT *p = Xs + row * a.I3 + k;
            if (row < row_end && kleft >= VE) x[j].load(p);
            else if (row < row_end && kleft > 0) x[j].load_some(p, int(kleft));
            else x[j].clear();
        }
    };
    auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < GROUPS; ++j) x[j].store(smem + buf * TILE + (gr + 32 * j) * SLAB_ROWB + gp * 16, nullptr);
    };
    fetch(0, 0);
    if constexpr (RAW)                                 // C, zero past its ends
        for (int i = tid; i < nk * 128; i += SLAB_THREADS) {
            const int row = i >> 3 & 15, k = (i >> 7) * KC + (i & 7) * VE;
            XGroup<FT, FT> c;
            c.load_some(Ch + row * a.I3 + k, row < a.J3 && k < a.I3 ? int(a.I3 - k) : 0);
            c.store(smem + 2 * TILE + ((i >> 7) * 16 + row) * SLAB_ROWB + (i & 7) * 16, nullptr);
        }
    store(0);
    __syncthreads();
    int buf = 0;
    for (int t = 0; t < ntiles; ++t) {
        wacc[0][0] = wacc[1][0] = zero_accv<accv>();
        const int64_t wrow0 = row_begin + int64_t(t) * SLAB_TM + wave * 32;
        for (int kc = 0; kc < nk; ++kc, buf ^= 1) {
            const bool last = kc + 1 == nk, more = !last || t + 1 < ntiles;
            if (more) fetch(last ? t + 1 : t, last ? 0 : kc + 1);
            if (wrow0 < row_end)
#pragma unroll
                for (int kg = 0; kg < 2; ++kg) {
                    const V16 c = RAW ? ld16(smem + 2 * TILE + (kc * 16 + l16) * SLAB_ROWB + kg * 64 + g * 16)
                                      : ld16(Ch + l16 * a.ldc + int64_t(kc) * KC + kg * KG + g * VE);
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb)
                        mma_kgroup<MATH>(wacc[mb][0], ld16(smem + buf * TILE + (wave * 32 + mb * 16 + l16) * SLAB_ROWB + kg * 64 + g * 16), c);
                }
            if (more) store(buf ^ 1);
            __syncthreads();
        }
        if (wrow0 >= row_end) continue;
        if (wrow0 + 32 > row_end)                      // (zeros times an infinite entry of C are NaN)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (wrow0 + mb * 16 + TR::acc_row(g, r) >= row_end) wacc[mb][0][r] = 0;
        if constexpr (RAW) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                const int64_t w0 = wrow0 + mb * 16, n = a.I2 - w0;
#pragma unroll
                for (int jb = 0; jb < JB; ++jb) {
                    const int64_t j = (jbase + jb) * 16 + l16;
                    const FT *b = Bh + (j < a.J2 ? j : a.J2 - 1) * a.I2 + w0;
                    FT bv[4];
                    if (MATH == M_F32 && n >= 16) __builtin_memcpy(bv, reinterpret_cast<const u32x4_u *>(b + 4 * g), 16);
                    else
#pragma unroll
                        for (int r = 0; r < 4; ++r) bv[r] = TR::acc_row(g, r) < n ? b[TR::acc_row(g, r)] : FT(0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if constexpr (MATH == M_F32) vacc[jb][0] = mfma_f32(bv[r], wacc[mb][0][r], vacc[jb][0]);
                        else vacc[jb][0] = mfma_f64(bv[r], wacc[mb][0][r], vacc[jb][0]);
                    }
                }
            }
        } else {
            slab_mode2<MATH, 2, 1, JB>(vacc, wacc, a, jbase, wrow0, l16, g);
        }
    }
    acc_t *Vp = static_cast<acc_t *>(a.V) + (i1 * a.P + (RAW ? s : s * 4 + wave)) * a.J2pad * a.J3pad + int64_t(jbase) * 16 * a.J3pad;
    if constexpr (RAW) {                               // the waves' shares, in order, where X was
        static_assert(4 * JB * 256 * sizeof(acc_t) <= 2 * TILE, "");
        acc_t *sum = reinterpret_cast<acc_t *>(smem);
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[(wave * JB + jb) * 256 + TR::acc_row(g, r) * 16 + l16] = vacc[jb][0][r];
        __syncthreads();
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
            const acc_t *v = sum + jb * 256 + tid;
            Vp[(jb * 16 + (tid >> 4)) * a.J3pad + (tid & 15)] = (v[0] + v[JB * 256]) + (v[2 * JB * 256] + v[3 * JB * 256]);
        }
    } else {
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r) Vp[(jb * 16 + TR::acc_row(g, r)) * a.J3pad + l16] = vacc[jb][0][r];
    }
}

// ---------------------------------------------------------------------------
// k_slab_dma: the same computation as k_slab for the common case where X is
// already in the operand format (bf16 X with bf16/bf16x3 arithmetic, f32 X
// with f32, f64 X with f64), rows are 16-byte aligned and I3 is a multiple of
// the 256-byte chunk.  X goes from HBM straight into LDS (global_load_lds,
// no register staging) in chunks of 128 rows x 256 bytes, double-buffered in
// two LDS arrays so that the compiler's wait before each barrier covers
// exactly the chunk about to be used.  Inside a chunk the 16-byte words of a
// row are XOR-swizzled by (row & 15): a 16-byte LDS read is served 16 lanes
// at a time over 64 banks (256 bytes), and the 16 rows of an operand
// fragment then land on 16 distinct 16-byte bank groups.  Chunks are 256
// bytes per row (64 KiB of LDS, two workgroups per compute unit).  Rows past
// the end of a slab range are read from a clamped (valid) row and their W
// rows zeroed before the mode-2 step.
// ---------------------------------------------------------------------------
template <int MATH, int WC, int NBW, int JB>
__global__ void __launch_bounds__(SLAB_THREADS, 2) k_slab_dma(const SlabArgs a) {
    typedef MathTraits<MATH> TR;
    typedef typename TR::lds_t LT;
    typedef typename TR::accv_t accv_t;
    typedef typename TR::acc_t acc_t;
    typedef typename TR::fac_t FT;
    constexpr int WR = 4 / WC, RW = SLAB_TM / WR, MB = RW / 16;
    constexpr int VE = TR::VE, KG = TR::KG;
    constexpr int ROWB = 256;                           // bytes of a row per chunk
    constexpr int KC = ROWB / int(sizeof(LT));         // k per chunk
    constexpr int NKG = ROWB / 64;                      // k-groups per chunk
    constexpr int STAGE = SLAB_TM * ROWB;
    constexpr int WPR = ROWB / 16;                      // 16-byte words per row
    constexpr int RPI = 1024 / ROWB;                    // rows per wave instruction
    constexpr int NDMA = SLAB_TM / 4 / RPI;             // instructions per wave per stage
    static_assert(MB >= 2 && MB % 2 == 0, "row blocks per wave");

    __shared__ __align__(1024) unsigned char st0[STAGE];
    __shared__ __align__(1024) unsigned char st1[STAGE];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave / WC, wc = wave % WC;
    const int l16 = lane & 15, g = lane >> 4;

    const int64_t i1 = blockIdx.x / a.S;
    const int s = int(blockIdx.x % a.S);
    const int64_t row_begin = int64_t(s) * a.rows_per_split;
    const int64_t row_end = a.I2 < row_begin + a.rows_per_split ? a.I2 : row_begin + a.rows_per_split;
    const int64_t nrows = row_end > row_begin ? row_end - row_begin : 0;
    const int64_t col0 = int64_t(blockIdx.y) * (WC * NBW * 16) + wc * NBW * 16;
    const int jbase = int(blockIdx.z) * JB;

    const LT *Xs = static_cast<const LT *>(a.X) + i1 * a.I2 * a.I3;
    const int64_t nk = a.I3 / KC;
    const int64_t ntiles = ceil_div(nrows, SLAB_TM);
    const int64_t nq = ntiles * nk;
    const FT *Ch = static_cast<const FT *>(a.Chi);
    const FT *Cl = static_cast<const FT *>(a.Clo);

    // DMA of chunk (t, kc) into one stage: wave w moves rows 32w .. 32w+31,
    // RPI rows per instruction; lane l fills slot (row, word l % WPR), which
    // holds logical word (l % WPR) ^ (row & 15) of that row.
    const int drow_in = lane / WPR, dpos = lane % WPR;
    auto dma = [&](unsigned char *stage, int64_t t, int64_t kc) {
        const int64_t r0 = row_begin + t * SLAB_TM;
#pragma unroll
        for (int j = 0; j < NDMA; ++j) {
            const int row = wave * 32 + RPI * j + drow_in;
            int64_t grow = r0 + row;
            grow = grow < row_end ? grow : row_end - 1;
            const int word = dpos ^ (row & 15);
            const LT *src = Xs + grow * a.I3 + kc * KC + word * VE;
            dma16_to_lds(src, stage + (wave * 32 + RPI * j) * ROWB);
        }
    };

    accv_t vacc[JB][NBW];
    accv_t wacc[MB][NBW];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) vacc[jb][nb] = zero_accv<accv_t>();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) wacc[mb][nb] = zero_accv<accv_t>();

    // one chunk of matrix-core work from a stage; the factor fragments of the
    // next k-group are loaded while the current one is on the matrix cores
    auto compute = [&](const unsigned char *stage, int64_t kc) {
        V16 bh[2][NBW], bl[2][NBW];
        auto load_c = [&](int slot, int kg) {
            const int64_t k0 = kc * KC + kg * KG + g * VE;
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                const int64_t off = (col0 + nb * 16 + l16) * a.ldc + k0;
                bh[slot][nb] = ld16(Ch + off);
                if constexpr (MATH == M_BF16X3) bl[slot][nb] = ld16(Cl + off);
            }
        };
        load_c(0, 0);
#pragma unroll
        for (int kg = 0; kg < NKG; ++kg) {
            if (kg + 1 < NKG) load_c((kg + 1) & 1, kg + 1);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int row = wr * RW + mb * 16 + l16;
                const int word = (kg * 4 + g) ^ (row & 15);
                V16 ah;
                ah.u = *reinterpret_cast<const u32x4 *>(stage + row * ROWB + word * 16);
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) {
                    mma_kgroup<MATH == M_BF16X3 ? M_BF16 : MATH>(wacc[mb][nb], ah, bh[kg & 1][nb]);
                    if constexpr (MATH == M_BF16X3) mma_kgroup<M_BF16>(wacc[mb][nb], ah, bl[kg & 1][nb]);
                }
            }
        }
    };
    // end of a 128-row tile: zero rows past the range, mode-2 step, reset W
    auto tile_end = [&](int64_t t) {
        const int64_t wrow0 = row_begin + t * SLAB_TM + wr * RW;
        if (row_begin + (t + 1) * SLAB_TM > row_end) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool dead = wrow0 + mb * 16 + TR::acc_row(g, r) >= row_end;
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb)
                        if (dead) wacc[mb][nb][r] = acc_t(0);
                }
        }
        slab_mode2<MATH, MB, NBW, JB>(vacc, wacc, a, jbase, wrow0, l16, g);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) wacc[mb][nb] = zero_accv<accv_t>();
    };

    int64_t t = 0, kc = 0;       // chunk being computed
    int64_t ft = 0, fkc = 0;     // chunk fetched next
    auto next = [&](int64_t &tt, int64_t &kk) { if (++kk == nk) { kk = 0; ++tt; } };
    if (nq > 0) {
        dma(st0, ft, fkc);
        next(ft, fkc);
    }
    for (int64_t q = 0; q < nq; q += 2) {
        __syncthreads();                       // chunk q is in st0; st1 is free
        if (q + 1 < nq) { dma(st1, ft, fkc); next(ft, fkc); }
        compute(st0, kc);
        if (kc == nk - 1) tile_end(t);
        next(t, kc);
        if (q + 1 >= nq) break;
        __syncthreads();                       // chunk q+1 is in st1; st0 is free
        if (q + 2 < nq) { dma(st0, ft, fkc); next(ft, fkc); }
        compute(st1, kc);
        if (kc == nk - 1) tile_end(t);
        next(t, kc);
    }

    acc_t *Vp = static_cast<acc_t *>(a.V) + (i1 * a.P + int64_t(s) * WR + wr) * a.J2pad * a.J3pad;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j2 = int64_t(jbase + jb) * 16 + TR::acc_row(g, r);
                Vp[j2 * a.J3pad + col0 + nb * 16 + l16] = vacc[jb][nb][r];
            }
}

// s_waitcnt with only the vector-memory count limited (gfx9 encoding:
// vmcnt bits [3:0] and [15:14], expcnt and lgkmcnt at their maxima).

// Mode-2 step for the bf16 forms with the B loads software-pipelined: W is
// first converted to its bf16 operand pairs (freeing the accumulators), then
// the tile's B fragments are taken in rounds of four 16-row blocks of j2 (hi
// and lo) over 32 rows, and the loads of round r + 1 are issued before the
// products of round r, so each round waits for loads that have had a round of
// products to land instead of a full L2 round trip.
template <int MATH, int MB, int NBW, int JB>
__device__ __forceinline__ void slab_mode2_pipe(typename MathTraits<MATH>::accv_t (&vacc)[JB][NBW],
                                                typename MathTraits<MATH>::accv_t (&wacc)[MB][NBW],
                                                const SlabArgs &a, int jbase, int64_t wrow0, int l16, int g) {
    static_assert(MATH == M_BF16 || MATH == M_BF16X3, "bf16 forms");
    constexpr bool X3 = MATH == M_BF16X3;
    constexpr int JG = JB < 4 ? JB : 4, NG = JB / JG, R = (MB / 2) * NG;
    const uint16_t *Bh = static_cast<const uint16_t *>(a.Bhi);
    const uint16_t *Bl = static_cast<const uint16_t *>(a.Blo);
    u32x4 wh[MB / 2][NBW], wl[MB / 2][NBW];
#pragma unroll
    for (int p = 0; p < MB / 2; ++p)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            const float v[8] = {wacc[2 * p][nb][0], wacc[2 * p][nb][1], wacc[2 * p][nb][2], wacc[2 * p][nb][3],
                                wacc[2 * p + 1][nb][0], wacc[2 * p + 1][nb][1], wacc[2 * p + 1][nb][2],
                                wacc[2 * p + 1][nb][3]};
            if constexpr (X3) bf16_split8(v, wh[p][nb], &wl[p][nb]);
            else wh[p][nb] = bf16_round8(v);
        }
    u32x4 bh[2][JG], bl[2][JG];
    auto load = [&](int r, int buf) __attribute__((always_inline)) {
        const int p = r / NG, j0 = (r % NG) * JG;
#pragma unroll
        for (int jj = 0; jj < JG; ++jj) {
            const int64_t off = int64_t((jbase + j0 + jj) * 16 + l16) * a.ldb + wrow0 + 32 * p + 8 * g;
            bh[buf][jj] = ld16(Bh + off).u;
            if constexpr (X3) bl[buf][jj] = ld16(Bl + off).u;
        }
    };
    load(0, 0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r + 1 < R) load(r + 1, (r + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        const int p = r / NG, j0 = (r % NG) * JG, cb = r & 1;
#pragma unroll
        for (int jj = 0; jj < JG; ++jj)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                auto &acc = vacc[j0 + jj][nb];
                acc = mfma_bf16(bh[cb][jj], wh[p][nb], acc);
                if constexpr (X3) {
                    acc = mfma_bf16(bh[cb][jj], wl[p][nb], acc);
                    acc = mfma_bf16(bl[cb][jj], wh[p][nb], acc);
                }
            }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---------------------------------------------------------------------------
// k_slab_lc: the slab kernel with the factor C staged through LDS, for bf16 X
// with the bf16 and bf16x3 forms where four waves share the columns (WC == 4).
//
// In the register-fed kernels every wave loads its own C fragments from L2
// for every k-group of every 128-row tile: twice the bytes of X, and each of
// those loads sits in the same in-order vector-memory queue as the X copies,
// so its wait can include a copy.  Here one workgroup per compute unit runs
// eight waves over 256-row tiles: the C chunk of the workgroup's columns (hi
// and lo) is copied into LDS by the same direct-to-LDS copies as X, once per
// workgroup and chunk, halving the C traffic, and the matrix-core waves read
// both operands from LDS.  Wave (wr, wc) owns rows 128 wr .. 128 wr + 127 of
// each tile and NBW column blocks.
//
// Chunks are 128 bytes of each row (64 values).  X has three LDS stages (two
// chunks in flight), C two (one chunk ahead: it comes from L2).  Copies are
// issued C(q+1) then X(q+2), so before the barrier of chunk q a wave waits
// until at most its copies of X(q+1) are outstanding (explicit vmcnt).  The
// stage reads are ds_read_b128 issued through inline assembly, waited for
// with explicit lgkmcnt waits that the fragments depend on: the compiler
// therefore never adds a wait of its own for the copies in flight, which it
// cannot tell apart by stage.  The 16-byte words of a 128-byte row are XOR-
// swizzled by (row >> 1) & 7: the 16 rows of a fragment read cover all 64
// banks.  At the end of a tile the mode-2 step copies B once per workgroup
// into the tile's consumed X and C stages (mode2_lds below) for all eight
// waves to read.  The two row halves' V partials are added through LDS at
// the end.
// ---------------------------------------------------------------------------
constexpr int LC_THREADS = 512;
constexpr int LC_XSTAGE = LC_TM * 128;               // 32 KiB

template <int OFF>
__device__ __forceinline__ u32x4 lds_read16_at(uint32_t addr) {
    static_assert(OFF >= 0 && OFF < 65536 && OFF % 16 == 0, "ds_read_b128 immediate offset");
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF) : "memory");
    return v;
}
// wait until at most N LDS reads of this wave are in flight
template <int N>
__device__ __forceinline__ void lds_wait() {
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N));
}
// makes r's value available only after the preceding wait (r was written by
// an LDS read issued through inline assembly)
__device__ __forceinline__ void lds_dep(u32x4 &r) { asm volatile("" : "+v"(r)); }
// Read order and waits of one chunk of k_slab_lc: per k-group NC C reads then
// MB X reads; group g = (kg, mb) needs reads up to need(g); before group g the
// reads up to issued(g) have been issued, keeping at most 12 in flight past
// the last read known to have returned.
template <int NC_, int MB, int NKG>
struct LcReadSched {
    static constexpr int NC = NC_, PER_KG = NC_ + MB, NR = NKG * PER_KG;
    static constexpr int need(int g) { return (g / MB) * PER_KG + NC + g % MB; }
    static constexpr int issued(int g) {
        if (g < 0) return 0;
        const int done = g == 0 ? 0 : need(g - 1) + 1;
        return done + 12 < NR ? done + 12 : NR;
    }
};
template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
// f(std::integral_constant<int, i>) for i = 0 .. N - 1, in order
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

template <int MATH, int NBW, int JB>
__global__ void __launch_bounds__(LC_THREADS, 1) k_slab_lc(const SlabArgs a) {
    typedef MathTraits<MATH> TR;
    typedef typename TR::accv_t accv_t;
    constexpr bool X3 = MATH == M_BF16X3;
    static_assert(MATH == M_BF16 || MATH == M_BF16X3, "bf16 forms");
    constexpr int WC = 4, RW = 128, MB = 8;
    constexpr int KC = 64, NKG = 2;                   // bf16 values per chunk row, k-groups per chunk
    constexpr int COLS = WC * NBW * 16;               // columns of the workgroup
    constexpr int CPART = COLS * 128;                 // bytes of one C part (hi or lo) per stage
    constexpr int CSTAGE = CPART * (X3 ? 2 : 1);
    constexpr int XOPS = LC_XSTAGE / 1024 / 8;        // X copy instructions per wave per chunk (4)
    constexpr int COPS = CSTAGE / 1024 / 8;           // C copy instructions per wave per chunk
    constexpr int NCF = NKG * NBW * (X3 ? 2 : 1);     // C fragments per chunk

    __shared__ __align__(1024) unsigned char xbuf[3 * LC_XSTAGE];
    __shared__ __align__(1024) unsigned char cbuf[2 * CSTAGE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WC, wc = wave % WC;
    const int l16 = lane & 15, g = lane >> 4;

    const int64_t i1 = blockIdx.x / a.S;
    const int s = int(blockIdx.x % a.S);
    const int64_t row_begin = int64_t(s) * a.rows_per_split;
    const int64_t row_end = a.I2 < row_begin + a.rows_per_split ? a.I2 : row_begin + a.rows_per_split;
    const int64_t nrows = row_end > row_begin ? row_end - row_begin : 0;
    const int64_t colb = int64_t(blockIdx.y) * COLS;  // first column of the workgroup
    const int jbase = int(blockIdx.z) * JB;
    const uint16_t *Xs = static_cast<const uint16_t *>(a.X) + i1 * a.I2 * a.I3;
    const uint16_t *Ch = static_cast<const uint16_t *>(a.Chi);
    const uint16_t *Cl = static_cast<const uint16_t *>(a.Clo);
    const int64_t nk = a.I3 / KC;
    const int64_t ntiles = ceil_div(nrows, LC_TM);
    const int64_t nq = ntiles * nk;

    // copies: 8 rows (or columns) of 128 bytes per instruction; lane l fills
    // word l % 8 of row l / 8 with logical word (l % 8) ^ ((row >> 1) & 7).
    // Addresses are a uniform base plus a 32-bit lane offset (the host
    // guarantees 256 rows of X, the columns of C and B each span less than 2 GiB);
    // X's lane offsets change only at a tile whose rows run past the range,
    // where rows are clamped to the last one.
    const int drow = lane >> 3, dpos = lane & 7;
    const int64_t xrow_bytes = a.I3 * 2, crow_bytes = a.ldc * 2;
    uint32_t xlo[XOPS], clo[COPS];
    const uint32_t xrow_b32 = uint32_t(xrow_bytes);
    auto set_x_offsets = [&](int64_t r0) __attribute__((always_inline)) {
        // last row of the range relative to the tile, at most LC_TM - 1
        const int64_t last64 = row_end - 1 - r0;
        const int last = __builtin_amdgcn_readfirstlane(int(last64 < LC_TM - 1 ? last64 : LC_TM - 1));
#pragma unroll
        for (int j = 0; j < XOPS; ++j) {
            const int row = (wave * XOPS + j) * 8 + drow;
            const uint32_t rr = uint32_t(row < last ? row : last);
            xlo[j] = rr * xrow_b32 + uint32_t((dpos ^ ((row >> 1) & 7)) << 4);
        }
    };
#pragma unroll
    for (int j = 0; j < COPS; ++j) {
        const int idx = wave * COPS + j;
        const int col = (idx % (COLS / 8)) * 8 + drow;
        clo[j] = uint32_t(col) * uint32_t(crow_bytes) + uint32_t((dpos ^ ((col >> 1) & 7)) << 4);
    }
    const char *xslab = reinterpret_cast<const char *>(Xs);
    const char *cbase[2] = {reinterpret_cast<const char *>(Ch + colb * a.ldc),
                            reinterpret_cast<const char *>((X3 ? Cl : Ch) + colb * a.ldc)};
    // stage arguments are LDS byte addresses
    auto copy_x = [&](uint32_t stage, int64_t t, int kc) __attribute__((always_inline)) {
        const char *base = xslab + (row_begin + t * LC_TM) * xrow_bytes + kc * 128;
#pragma unroll
        for (int j = 0; j < XOPS; ++j) dma16s_to_lds_m0(base, xlo[j], stage + uint32_t((wave * XOPS + j) * 8 * 128));
    };
    auto copy_c = [&](uint32_t stage, int kc) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < COPS; ++j) {
            const int idx = wave * COPS + j;
            const int part = idx / (COLS / 8);         // 0: hi, 1: lo
            const int col0 = (idx % (COLS / 8)) * 8;
            dma16s_to_lds_m0(cbase[part] + kc * 128, clo[j], stage + uint32_t(part * CPART + col0 * 128));
        }
    };

    accv_t vacc[JB][NBW];
    accv_t wacc[MB][NBW];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) vacc[jb][nb] = zero_accv<accv_t>();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) wacc[mb][nb] = zero_accv<accv_t>();

    // per-lane LDS byte offsets of the fragment words of k-group kg: the
    // swizzle key (row >> 1) & 7 of rows 16 m + l16 is (l16 >> 1) & 7 for
    // every 16-row block, so block m adds the immediate m * 2048
    uint32_t xl[NKG], cl[NKG];
#pragma unroll
    for (int kg = 0; kg < NKG; ++kg) {
        const uint32_t w = uint32_t(((kg * 4 + g) ^ ((l16 >> 1) & 7)) << 4);
        xl[kg] = uint32_t((wr * RW + l16) * 128) + w;
        cl[kg] = uint32_t((wc * NBW * 16 + l16) * 128) + w;
    }
    const uint32_t xlds = lds_offset(xbuf), clds = lds_offset(cbuf);

    // one chunk of matrix-core work, in groups (k-group kg, 16-row block mb).
    // The chunk's LDS reads are issued in the order the groups consume them
    // (per k-group: its C fragments, then the X fragments of blocks 0 .. MB-1)
    // with at most 12 in flight (the LDS counter counts to 15; 12 keeps the
    // fragments within the registers at two waves per SIMD), and each group
    // waits only until its own operands have returned (LDS reads of a wave
    // return in order): the first products start after a few reads instead of
    // after all of them.
    typedef LcReadSched<NCF / NKG, MB, NKG> SC;
    auto compute = [&](uint32_t xs, uint32_t cs, auto &&after_group) __attribute__((always_inline)) {
        u32x4 rd[SC::NR];
        const uint32_t xa[NKG] = {xs + xl[0], xs + xl[1]};
        const uint32_t ca[NKG] = {cs + cl[0], cs + cl[1]};
        auto issue = [&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value, kg = i / SC::PER_KG, w = i % SC::PER_KG;
            if constexpr (w < SC::NC) {
                constexpr int nb = w / (X3 ? 2 : 1), part = w % (X3 ? 2 : 1);
                rd[i] = lds_read16_at<part * CPART + nb * 2048>(ca[kg]);
            } else {
                rd[i] = lds_read16_at<(w - SC::NC) * 2048>(xa[kg]);
            }
        };
        static_for<NKG * MB>([&](auto G) __attribute__((always_inline)) {
            constexpr int g = decltype(G)::value, kg = g / MB, mb = g % MB;
            constexpr int i0 = SC::issued(g - 1), i1 = SC::issued(g);
            static_for<i1 - i0>([&](auto J) __attribute__((always_inline)) {
                issue(std::integral_constant<int, i0 + decltype(J)::value>{});
            });
            lds_wait<i1 - SC::need(g) - 1>();
            constexpr int cb = kg * SC::PER_KG, xr = cb + SC::NC + mb;
            lds_dep(rd[xr]);
            if constexpr (mb == 0)
                static_for<SC::NC>([&](auto C) __attribute__((always_inline)) { lds_dep(rd[cb + decltype(C)::value]); });
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                wacc[mb][nb] = mfma_bf16(rd[xr], rd[cb + nb * (X3 ? 2 : 1)], wacc[mb][nb]);
                if constexpr (X3) wacc[mb][nb] = mfma_bf16(rd[xr], rd[cb + nb * 2 + 1], wacc[mb][nb]);
            }
            after_group(G);
        });
    };
    // Mode-2 step of a tile with B staged through LDS.  The four column waves
    // of a row half need the same B fragments; copied once per workgroup,
    // B costs a quarter of the L2 reads of per-wave loads, and the copies of
    // several phases are in flight at once.  A phase is one k-step of 32 rows
    // in each half (the W pairs p) for JP 16-row blocks of j2: B[j2][32 rows]
    // of both halves, hi (and lo), 64 bytes per j2 row with the 16-byte
    // pieces XOR-swizzled by (j2 row >> 2) & 3.  The buffers are the X and C
    // stages of the tile's last chunk, free once every wave has consumed
    // them; NBUF - 1 phases are in flight ahead of the one being multiplied.
    constexpr int PARTS = X3 ? 2 : 1;
    constexpr int JP = JB < 4 ? JB : 4;                  // j2 blocks per phase
    constexpr bool LDS_B = PARTS * JP >= 4;              // whole copy instructions per wave
    constexpr int PB = PARTS * JP * 2048;                // bytes per phase
    constexpr int XB = LC_XSTAGE / PB, CB = CSTAGE / PB; // phase buffers in an X / a C stage
    constexpr int NBUF = XB + CB < 4 ? XB + CB : 4;
    constexpr int NJH = JB / JP, NPH = (MB / 2) * NJH;
    constexpr int CPB = LDS_B ? PARTS * 2 * JP / 8 : 1;  // copy instructions per wave and phase
    static_assert(!LDS_B || (NBUF >= 2 && XB * PB == LC_XSTAGE && CB >= 1 && 8 * CPB == PARTS * 2 * JP),
                  "mode-2 phase buffers");
    // copy instruction k of this wave fills phase rows 16 i .. 16 i + 15 with
    // i = wave + 8 k: part i / (2 JP), half (i / JP) % 2, j2 rows (i % JP) * 16 +
    // lane / 4; lane l loads logical piece (l % 4) ^ ((row >> 2) & 3)
    uint32_t bofs[CPB];
    {
        const int r = lane >> 2, piece = (lane & 3) ^ ((r >> 2) & 3);
#pragma unroll
        for (int k = 0; k < CPB; ++k) {
            const int i = wave + 8 * k;
            bofs[k] = uint32_t((jbase * 16 + (i % JP) * 16 + r) * a.ldb * 2 + piece * 16);
        }
    }
    // per-lane LDS offset of the B fragment words: row wr * JP * 16 + l16
    const uint32_t brd = uint32_t((wr * JP * 16 + l16) * 64 + ((g ^ ((l16 >> 2) & 3)) << 4));
    auto mode2_lds = [&](int64_t t, bool live, uint32_t xs_done, uint32_t cs_done) __attribute__((always_inline)) {
        constexpr int PAIRS = MB / 2;
        u32x4 wh[PAIRS][NBW], wl[PAIRS][NBW];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                const float v[8] = {wacc[2 * p][nb][0], wacc[2 * p][nb][1], wacc[2 * p][nb][2], wacc[2 * p][nb][3],
                                    wacc[2 * p + 1][nb][0], wacc[2 * p + 1][nb][1], wacc[2 * p + 1][nb][2],
                                    wacc[2 * p + 1][nb][3]};
                if constexpr (X3) bf16_split8(v, wh[p][nb], &wl[p][nb]);
                else wh[p][nb] = bf16_round8(v);
            }
        // byte column of each half's rows in B; a half past the range copies
        // (and ignores) columns 0..127, which exist in every row of B
        const int64_t hb = row_begin + t * LC_TM;
        const uint32_t colb[2] = {uint32_t(hb * 2), hb + RW < row_end ? uint32_t((hb + RW) * 2) : 0u};
        const char *bsrc[2] = {static_cast<const char *>(a.Bhi), static_cast<const char *>(X3 ? a.Blo : a.Bhi)};
        auto buf = [&](int b) __attribute__((always_inline)) -> uint32_t {
            return b < XB ? xs_done + uint32_t(b * PB) : cs_done + uint32_t((b - XB) * PB);
        };
        auto issue = [&](auto PH) __attribute__((always_inline)) {
            constexpr int ph = decltype(PH)::value, p = ph / NJH, jh = ph % NJH;
            const uint32_t dst = buf(ph % NBUF);
#pragma unroll
            for (int k = 0; k < CPB; ++k) {
                const int i = wave + 8 * k;
                const char *src = bsrc[i / (2 * JP)] + colb[(i / JP) & 1] + int64_t(jh * JP * 16) * a.ldb * 2 + 64 * p;
                dma16s_to_lds_m0(src, bofs[k], dst + uint32_t(i * 1024));
            }
        };
        // every wave has consumed the chunk's X and C stages
        __builtin_amdgcn_s_barrier();
        static_for<NBUF - 1>([&](auto I) __attribute__((always_inline)) {
            if constexpr (decltype(I)::value < NPH) issue(I);
        });
        static_for<NPH>([&](auto PH) __attribute__((always_inline)) {
            constexpr int ph = decltype(PH)::value, p = ph / NJH, jh = ph % NJH;
            constexpr int last = ph + NBUF - 2 < NPH - 1 ? ph + NBUF - 2 : NPH - 1;
            // this wave's copies of phase ph (and of everything issued
            // before them) have landed; after the barrier, every wave's have,
            // and every wave is done with phase ph - 1's buffer
            wait_vmcnt<CPB * (last - ph)>();
            __builtin_amdgcn_s_barrier();
            if constexpr (ph + NBUF - 1 < NPH) issue(std::integral_constant<int, ph + NBUF - 1>{});
            if (live) {
                const uint32_t ba = buf(ph % NBUF) + brd;
                u32x4 fr[JP][PARTS];
                static_for<JP * PARTS>([&](auto R) __attribute__((always_inline)) {
                    constexpr int rr = decltype(R)::value, jj = rr / PARTS, part = rr % PARTS;
                    fr[jj][part] = lds_read16_at<part * JP * 2048 + jj * 1024>(ba);
                });
                static_for<JP>([&](auto JJ) __attribute__((always_inline)) {
                    constexpr int jj = decltype(JJ)::value;
                    lds_wait<(JP - 1 - jj) * PARTS>();
                    lds_dep(fr[jj][0]);
                    if constexpr (X3) lds_dep(fr[jj][PARTS - 1]);
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) {
                        auto &acc = vacc[jh * JP + jj][nb];
                        acc = mfma_bf16(fr[jj][0], wh[p][nb], acc);
                        if constexpr (X3) {
                            acc = mfma_bf16(fr[jj][0], wl[p][nb], acc);
                            acc = mfma_bf16(fr[jj][PARTS - 1], wh[p][nb], acc);
                        }
                    }
                });
            }
        });
    };
    auto tile_end = [&](int64_t t, uint32_t xs_done, uint32_t cs_done) __attribute__((always_inline)) {
        const int64_t wrow0 = row_begin + t * LC_TM + wr * RW;
        // a row half that starts past the range (the upper half of a partial
        // last tile) contributes nothing and reads no B: its columns could lie
        // past the padded row stride of B, which is a multiple of 128 only
        const bool live = wrow0 < row_end;
        if (live && wrow0 + RW > row_end) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool dead = wrow0 + mb * 16 + TR::acc_row(g, r) >= row_end;
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb)
                        if (dead) wacc[mb][nb][r] = 0.f;
                }
        }
        // rows past the range in this half contribute zeros; B's padded
        // columns up to the next multiple of 128 are zeros
        if constexpr (LDS_B) {
            mode2_lds(t, live, xs_done, cs_done);
        } else {
            if (live) slab_mode2_pipe<MATH, MB, NBW, JB>(vacc, wacc, a, jbase, wrow0, l16, g);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) wacc[mb][nb] = zero_accv<accv_t>();
    };

    // chunk q = t nk + kc: tile t, k-chunk kc.  The copies run ahead of the
    // work: X two chunks (coordinates tx, kx), C one chunk (kcn).  C's copies
    // are issued right after the barrier; X's are spread between the
    // matrix-core groups of the chunk (one after every second group), so that
    // a wave whose copy waits for room in the memory pipeline has products in
    // flight.
    const int nkc = int(nk);
    int64_t tx = 0;
    int kx = 0, kcn = 0;
    auto next_c = [&](uint32_t stage) __attribute__((always_inline)) {
        copy_c(stage, kcn);
        if (++kcn == nkc) kcn = 0;
    };
    static_assert(2 * XOPS <= NKG * MB, "one X copy per two groups");
    if (nq > 0) {
        set_x_offsets(row_begin);
        copy_x(xlds, 0, 0);
        next_c(clds);
        if (nq > 1) {
            if (nkc == 1) set_x_offsets(row_begin + LC_TM);
            copy_x(xlds + LC_XSTAGE, nkc == 1 ? 1 : 0, nkc == 1 ? 0 : 1);
        }
        tx = nkc <= 2 ? (nkc == 1 ? 2 : 1) : 0;
        kx = nkc <= 2 ? 0 : 2;
    }
    int64_t t = 0;
    int kc = 0, xst = 0, cst = 0;
    for (int64_t q = 0; q < nq; ++q) {
        // chunk q landed everywhere: this wave's copies of X(q) and C(q) are
        // done when at most its copies of X(q + 1) are outstanding
        if (q + 1 < nq) wait_vmcnt<XOPS>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        if (q + 1 < nq) next_c(clds + uint32_t((cst ^ 1) * CSTAGE));
        const bool x_next = q + 2 < nq, last_of_tile = kc == nkc - 1;
        const uint32_t xstage = xlds + uint32_t((xst == 0 ? 2 : xst - 1) * LC_XSTAGE);
        const char *xb = xslab;
        if (x_next) {
            if (kx == 0) set_x_offsets(row_begin + tx * LC_TM);
            xb = xslab + (row_begin + tx * LC_TM) * xrow_bytes + kx * 128;
        }
        const uint32_t xs = xlds + uint32_t(xst * LC_XSTAGE), cs = clds + uint32_t(cst * CSTAGE);
        compute(xs, cs, [&](auto G) __attribute__((always_inline)) {
            constexpr int g = decltype(G)::value;
            if constexpr (g % 2 == 1 && g / 2 < XOPS)
                if (x_next) dma16s_to_lds_m0(xb, xlo[g / 2], xstage + uint32_t((wave * XOPS + g / 2) * 1024));
        });
        if (last_of_tile) {
            tile_end(t, xs, cs);
            kc = 0;
            ++t;
        } else {
            ++kc;
        }
        if (x_next && ++kx == nkc) { kx = 0; ++tx; }
        xst = xst == 2 ? 0 : xst + 1;
        cst ^= 1;
    }

    // the upper row half adds its V partial to the lower one's through LDS
    // (every chunk has been consumed: the X stages are free)
    constexpr int NV = JB * NBW * 4;
    constexpr int PER_STAGE = LC_XSTAGE / 4 / 256;  // floats of one (wc, lane) slot per stage
    static_assert(NV <= 2 * PER_STAGE, "reduction buffer");
    __syncthreads();
    auto slot = [&](int v) __attribute__((always_inline)) -> float * {   // v-th value of this (wc, lane)
        float *base = reinterpret_cast<float *>(xbuf + (v < PER_STAGE ? 0 : LC_XSTAGE));
        return base + ((v % PER_STAGE) * 4 + wc) * 64 + lane;
    };
    if (wr == 1) {
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) *slot((jb * NBW + nb) * 4 + r) = vacc[jb][nb][r];
    }
    __syncthreads();
    if (wr != 0) return;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r) vacc[jb][nb][r] += *slot((jb * NBW + nb) * 4 + r);

    float *Vp = static_cast<float *>(a.V) + (i1 * a.P + s) * a.J2pad * a.J3pad;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j2 = int64_t(jbase + jb) * 16 + TR::acc_row(g, r);
                Vp[j2 * a.J3pad + colb + wc * NBW * 16 + nb * 16 + l16] = vacc[jb][nb][r];
            }
}

// ---------------------------------------------------------------------------
// Mode-1 contraction with partial sums:
//   Y[j1, n] = sum_i1 A[j1, i1] * sum_p V[i1][p][n],   n = j2 * J3pad + j3.
// A workgroup owns 64 columns n and up to 128 rows j1 (grid.z tiles larger
// J1); grid.y splits the i1 range.  V is streamed once:
// each lane reads one column over VE consecutive rows (a wave reads 256
// contiguous bytes per row), converts to the operand format and stores the
// VE values as one 16-byte LDS word, k-contiguous, which is exactly the
// k-slot fragment the B operand wants.  With one split the result goes to Y;
// otherwise to per-split partials summed by k_mode1_reduce.
// ---------------------------------------------------------------------------
struct Mode1Args {
    const void *Ahi, *Alo;   // [J1pad][lda]; in float and double the caller's A (lda = I1)
    int64_t lda;
    const void *V;           // [I1][P][NN]
    int64_t I1;
    int P;
    int64_t NN, J3pad;
    void *Y;                 // final output, used when KS == 1
    void *Ypart;             // [KS][J1pad][NN] partials, used when KS > 1
    int64_t J1, J2, J3, J1pad;
    int KS;
    int64_t rows_per_split;
};

template <int MATH>
struct Mode1Cfg {
    typedef MathTraits<MATH> TR;
    typedef typename TR::lds_t LT;
    static constexpr int VE = TR::VE, KG = TR::KG;
    static constexpr int KT = 2 * KG;                                  // rows per chunk
    static constexpr int ROWB = KT * int(sizeof(LT)) + 16;             // LDS stride per column
    static constexpr int BUFB = 64 * ROWB;
    static constexpr int ITEMS = KT * 64 / (256 * VE);                 // 16-byte words per thread per chunk
    static constexpr bool SPLIT = (MATH == M_BF16X3);
};

// A's fragment for 16 rows from m on, k slots k .. k + VE - 1 of lane group g:
// the padded operand array, or in float and double the caller's factor (rows
// past J1 repeat the last one and are not stored; place_a() once the fragment
// is needed, where the k range passes I1).
template <int MATH>
__device__ __forceinline__ void fetch_a(const Mode1Args &a, const void *A, int64_t m, int64_t k,
                                        XGroup<typename MathTraits<MATH>::fac_t, typename MathTraits<MATH>::fac_t> &f) {
    typedef typename MathTraits<MATH>::fac_t FT;
    if constexpr (MATH == M_F32 || MATH == M_F64) {
        // (an A shorter than a group is read by place_a(): here V, unused)
        const int64_t total = a.J1 * a.I1, VE = MathTraits<MATH>::VE, wide = total < VE ? 0 : total - VE;
        const FT *base = static_cast<const FT *>(total < VE ? a.V : A);
        const int64_t off = (m < a.J1 ? m : a.J1 - 1) * a.I1 + (k < a.I1 ? k : 0);
        f.load(base + (off < wide ? off : wide));
    } else {
        f.raw = ld16(static_cast<const FT *>(A) + m * a.lda + k);
    }
}
template <int MATH>
__device__ __forceinline__ void place_a(const Mode1Args &a, int64_t m, int64_t k,
                                        XGroup<typename MathTraits<MATH>::fac_t, typename MathTraits<MATH>::fac_t> &f) {
    if constexpr (MATH == M_F32 || MATH == M_F64) {
        const int64_t left = a.I1 - k;
        const int n = left >= MathTraits<MATH>::VE ? MathTraits<MATH>::VE : (left > 0 ? int(left) : 0);
        place_group(f, static_cast<const typename MathTraits<MATH>::fac_t *>(a.Ahi),
                    (m < a.J1 ? m : a.J1 - 1) * a.I1 + (n > 0 ? k : 0), a.J1 * a.I1, n);
    }
}

// MW 16-row blocks and NW 16-column blocks per wave.  NW == 4: the waves
// split the rows (wave w: blocks w*MW ..), each covering all 64 columns, so
// every element of A is fetched once per workgroup; NW == 1: the waves split
// the columns (small J1).
template <int MATH, int MW, int NW>
__global__ void __launch_bounds__(256) k_mode1(const Mode1Args a) {
    typedef Mode1Cfg<MATH> CF;
    typedef MathTraits<MATH> TR;
    typedef typename TR::accv_t accv_t;
    typedef typename TR::acc_t acc_t;
    typedef typename TR::fac_t FT;
    constexpr int VE = CF::VE, KG = CF::KG, KT = CF::KT, ITEMS = CF::ITEMS;
    __shared__ __align__(16) unsigned char lds[2 * CF::BUFB * (CF::SPLIT ? 2 : 1)];
    unsigned char *lhi = lds, *llo = lds + 2 * CF::BUFB;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t n0 = int64_t(blockIdx.x) * 64;
    const int ks = int(blockIdx.y);
    const int64_t kb = int64_t(ks) * a.rows_per_split;
    const int64_t ke = a.I1 < kb + a.rows_per_split ? a.I1 : kb + a.rows_per_split;
    const int64_t nch = ke > kb ? ceil_div(ke - kb, KT) : 0;
    const acc_t *V = static_cast<const acc_t *>(a.V);
    const FT *Ah = static_cast<const FT *>(a.Ahi);
    const FT *Al = static_cast<const FT *>(a.Alo);

    // loader: thread (column c = tid % 64, word w = tid / 64 + 4*item) covers rows VE*w .. VE*w+VE-1
    const int lc = tid & 63, lw = tid >> 6;
    // V chunks in flight in registers: two ahead of the one being computed
    // (slots ch % 2), one ahead for bf16x3 with two row blocks per wave.  The
    // last partial of V is added when the chunk is stored, not when it is
    // fetched, so that its trip (with one partial, all of them) is under way
    // during the products.
    struct Chunk { acc_t sum[ITEMS][VE], last[ITEMS][VE]; } pre2[2];
    // all ITEMS*VE loads of one partial are independent and issued together;
    // rows past the range read row kb (valid) and are zeroed
    auto fetch = [&](int64_t ch, Chunk &c) __attribute__((always_inline)) {
        const int64_t r0 = kb + ch * KT;
        auto load = [&](int p, acc_t (&dst)[ITEMS][VE]) __attribute__((always_inline)) {
            const acc_t *vp = V + int64_t(p) * a.NN + n0 + lc;
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
#pragma unroll
                for (int e = 0; e < VE; ++e) {
                    const int64_t k = r0 + (lw + 4 * it) * VE + e;
                    dst[it][e] = vp[(k < ke ? k : kb) * a.P * a.NN];
                }
            __builtin_amdgcn_sched_barrier(0);   // (else the scheduler may issue them one by one to save registers)
        };
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
#pragma unroll
            for (int e = 0; e < VE; ++e) c.sum[it][e] = acc_t(0);
        for (int p = 0; p < a.P - 1; ++p) {
            acc_t t[ITEMS][VE];
            load(p, t);
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
#pragma unroll
                for (int e = 0; e < VE; ++e) c.sum[it][e] += t[it][e];
        }
        load(a.P - 1, c.last);
    };
    auto store = [&](int64_t ch, int buf, Chunk &c) __attribute__((always_inline)) {
        const int64_t r0 = kb + ch * KT;
        acc_t pre[ITEMS][VE];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
#pragma unroll
            for (int e = 0; e < VE; ++e) pre[it][e] = c.sum[it][e] + c.last[it][e];
        if (r0 + KT > ke)
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
#pragma unroll
                for (int e = 0; e < VE; ++e)
                    if (r0 + (lw + 4 * it) * VE + e >= ke) pre[it][e] = acc_t(0);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int off = buf * CF::BUFB + lc * CF::ROWB + (lw + 4 * it) * 16;
            if constexpr (MATH == M_F32) {
                *reinterpret_cast<f32x4 *>(lhi + off) = f32x4{pre[it][0], pre[it][1], pre[it][2], pre[it][3]};
            } else if constexpr (MATH == M_F64) {
                *reinterpret_cast<f64x2 *>(lhi + off) = f64x2{pre[it][0], pre[it][1]};
            } else {
                const float v[8] = {pre[it][0], pre[it][1], pre[it][2], pre[it][3],
                                    pre[it][4], pre[it][5], pre[it][6], pre[it][7]};
                u32x4 h, l;
                if constexpr (CF::SPLIT) {
                    bf16_split8(v, h, &l);
                    *reinterpret_cast<u32x4 *>(llo + off) = l;
                } else {
                    h = bf16_round8(v);
                }
                *reinterpret_cast<u32x4 *>(lhi + off) = h;
            }
        }
    };

    constexpr int MBW = NW == 4 ? 4 * MW : MW;          // 16-row blocks per workgroup
    const int mbase = NW == 4 ? wave * MW : 0;
    const int nbase = NW == 4 ? 0 : wave;
    const int64_t m0 = int64_t(blockIdx.z) * MBW * 16;
    accv_t acc[MW][NW];
#pragma unroll
    for (int i = 0; i < MW; ++i)
#pragma unroll
        for (int j = 0; j < NW; ++j) acc[i][j] = zero_accv<accv_t>();

    // A's fragments of a chunk are loaded one chunk ahead and before the next
    // chunk's V prefetch: vector-memory loads complete in order, so a wait for
    // A issued after the prefetch would also wait for the prefetch's HBM trip
    XGroup<FT, FT> fah[MW][2], fal[MW][2];
    auto load_a = [&](int64_t ch) __attribute__((always_inline)) {
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) {
            const int64_t k0 = kb + ch * KT + kg * KG + g * VE;
#pragma unroll
            for (int i = 0; i < MW; ++i) {
                const int64_t m = m0 + (mbase + i) * 16 + l16;
                fetch_a<MATH>(a, Ah, m, k0, fah[i][kg]);
                if constexpr (CF::SPLIT) fetch_a<MATH>(a, Al, m, k0, fal[i][kg]);
            }
        }
    };
    auto compute = [&](int64_t ch, int buf) __attribute__((always_inline)) {
        if constexpr (MATH == M_F32 || MATH == M_F64) if (kb + (ch + 1) * KT > a.I1) {
#pragma unroll
            for (int kg = 0; kg < 2; ++kg)
#pragma unroll
                for (int i = 0; i < MW; ++i)
                    place_a<MATH>(a, m0 + (mbase + i) * 16 + l16, kb + ch * KT + kg * KG + g * VE, fah[i][kg]);
        }
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) {
            V16 bh[NW], bl[NW];
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const int loff = buf * CF::BUFB + ((nbase + j) * 16 + l16) * CF::ROWB + kg * 64 + g * 16;
                bh[j].u = *reinterpret_cast<const u32x4 *>(lhi + loff);
                if constexpr (CF::SPLIT) bl[j].u = *reinterpret_cast<const u32x4 *>(llo + loff);
            }
#pragma unroll
            for (int i = 0; i < MW; ++i) {
                const V16 ah = fah[i][kg].raw;
                V16 al;
                if constexpr (CF::SPLIT) al = fal[i][kg].raw;
#pragma unroll
                for (int j = 0; j < NW; ++j) {
                    mma_kgroup<MATH == M_BF16X3 ? M_BF16 : MATH>(acc[i][j], ah, bh[j]);
                    if constexpr (CF::SPLIT) {
                        mma_kgroup<M_BF16>(acc[i][j], ah, bl[j]);
                        mma_kgroup<M_BF16>(acc[i][j], al, bh[j]);
                    }
                }
            }
        }
    };
    // one chunk: prefetch chunk ch + 2 into the slot chunk ch left, compute
    // chunk ch, then store chunk ch + 1 (slot 1 - S) and load its A fragments
    auto step = [&](int64_t ch, auto SLOT) __attribute__((always_inline)) {
        constexpr int S = decltype(SLOT)::value;
        if (ch + 2 < nch) fetch(ch + 2, pre2[S]);
        compute(ch, S);
        if (ch + 1 < nch) {
            store(ch + 1, 1 - S, pre2[1 - S]);
            load_a(ch + 1);
        }
        __syncthreads();
    };
    if constexpr (CF::SPLIT && MW == 2) {
        // bf16x3 with two row blocks per wave: one chunk ahead (two would take
        // the registers of a third resident wave per SIMD, measured slower)
        if (nch > 0) {
            fetch(0, pre2[0]);
            store(0, 0, pre2[0]);
            load_a(0);
        }
        __syncthreads();
        for (int64_t ch = 0; ch < nch; ++ch) {
            if (ch + 1 < nch) fetch(ch + 1, pre2[0]);
            compute(ch, int(ch & 1));
            if (ch + 1 < nch) {
                store(ch + 1, int((ch + 1) & 1), pre2[0]);
                load_a(ch + 1);
            }
            __syncthreads();
        }
    } else {
        if (nch > 0) {
            fetch(0, pre2[0]);
            if (nch > 1) fetch(1, pre2[1]);
            store(0, 0, pre2[0]);
            load_a(0);
        }
        __syncthreads();
        for (int64_t ch = 0; ch < nch; ch += 2) {
            step(ch, std::integral_constant<int, 0>{});
            if (ch + 1 < nch) step(ch + 1, std::integral_constant<int, 1>{});
        }
    }

    acc_t *Y = static_cast<acc_t *>(a.Y);
    acc_t *Yp = static_cast<acc_t *>(a.Ypart) + int64_t(ks) * a.J1pad * a.NN;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const int64_t n = n0 + (nbase + j) * 16 + l16;
        const int64_t j2 = n / a.J3pad, j3 = n % a.J3pad;
#pragma unroll
        for (int i = 0; i < MW; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j1 = m0 + (mbase + i) * 16 + TR::acc_row(g, r);
                if (a.KS == 1) {
                    if (j1 < a.J1 && j2 < a.J2 && j3 < a.J3) Y[(j1 * a.J2 + j2) * a.J3 + j3] = acc[i][j][r];
                } else {
                    Yp[j1 * a.NN + n] = acc[i][j][r];
                }
            }
    }
}

// The same contraction in one launch where V is small: a workgroup owns 16
// columns n and MW blocks of 16 rows j1; its NW waves share the i1 range by
// k-groups (wave w: groups w, w + NW, ...), read V and A straight into operand
// registers, and their sums meet in LDS, in order.  Every load of a wave's
// first groups is in flight at once and there is no split to sum in a second
// launch.  Bound by the trips to V and A; 64^3 -> 16^3 in double: k_mode1 and
// k_mode1_reduce 4.2 + 2.4 us and a launch, now 3.4 us; chains, k_mode1 first: 232
// x 136 x 264 -> 104 x 43 x 80 in float (V 11 MB) 82 and 66 us, 512^3 -> 64 in
// float (V 16 MB) 218 and 215; at 1024 x 512 x 512 -> 128 in bf16x3 (V 64 MB)
// 231 and 278.
template <int MATH, int MW, int NW>
__global__ void __launch_bounds__(64 * NW) k_mode1_small(const Mode1Args a) {
    typedef Mode1Cfg<MATH> CF;
    typedef MathTraits<MATH> TR;
    typedef typename TR::accv_t accv_t;
    typedef typename TR::acc_t acc_t;
    typedef typename TR::fac_t FT;
    constexpr int VE = CF::VE, KG = CF::KG;
    constexpr bool X3 = CF::SPLIT;
    __shared__ acc_t red[NW][MW * 4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int64_t n = int64_t(blockIdx.x) * 16 + l16, m0 = int64_t(blockIdx.z) * MW * 16;
    const acc_t *V = static_cast<const acc_t *>(a.V) + n;
    accv_t acc[MW];
#pragma unroll
    for (int i = 0; i < MW; ++i) acc[i] = zero_accv<accv_t>();
    const int64_t ng = ceil_div(a.I1, KG);
    for (int64_t q = wave; q < ng; q += NW) {
        const int64_t k = q * KG + g * VE;
        XGroup<FT, FT> ah[MW], al[MW];
#pragma unroll
        for (int i = 0; i < MW; ++i) {
            fetch_a<MATH>(a, a.Ahi, m0 + i * 16 + l16, k, ah[i]);
            if constexpr (X3) fetch_a<MATH>(a, a.Alo, m0 + i * 16 + l16, k, al[i]);
        }
        acc_t v[VE];
#pragma unroll
        for (int e = 0; e < VE; ++e) v[e] = acc_t(0);
        auto add = [&](int p, auto NP) __attribute__((always_inline)) {
            constexpr int N = decltype(NP)::value;
            acc_t t[N][VE];
#pragma unroll
            for (int b = 0; b < N; ++b)
#pragma unroll
                for (int e = 0; e < VE; ++e) t[b][e] = V[((k + e < a.I1 ? k + e : a.I1 - 1) * a.P + p + b) * a.NN];
#pragma unroll
            for (int b = 0; b < N; ++b)
#pragma unroll
                for (int e = 0; e < VE; ++e) v[e] += t[b][e];
        };
        int p = 0;
        for (; p + 4 <= a.P; p += 4) add(p, std::integral_constant<int, 4>{});
        for (; p + 2 <= a.P; p += 2) add(p, std::integral_constant<int, 2>{});
        if (p < a.P) add(p, std::integral_constant<int, 1>{});
        if ((q + 1) * KG > a.I1) {
#pragma unroll
            for (int e = 0; e < VE; ++e) v[e] = k + e < a.I1 ? v[e] : acc_t(0);
#pragma unroll
            for (int i = 0; i < MW; ++i) place_a<MATH>(a, m0 + i * 16 + l16, k, ah[i]);
        }
        V16 bh, bl;
        if constexpr (MATH == M_F32) {
            bh.u = __builtin_bit_cast(u32x4, f32x4{v[0], v[1], v[2], v[3]});
        } else if constexpr (MATH == M_F64) {
            bh.d[0] = v[0];
            bh.d[1] = v[1];
        } else {
            const float f[8] = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
            if constexpr (X3) bf16_split8(f, bh.u, &bl.u);
            else bh.u = bf16_round8(f);
        }
#pragma unroll
        for (int i = 0; i < MW; ++i) {
            mma_kgroup<X3 ? M_BF16 : MATH>(acc[i], ah[i].raw, bh);
            if constexpr (X3) {
                mma_kgroup<M_BF16>(acc[i], ah[i].raw, bl);
                mma_kgroup<M_BF16>(acc[i], al[i].raw, bh);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < MW; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][i * 4 + r][lane] = acc[i][r];
    __syncthreads();
    const int64_t j2 = n / a.J3pad, j3 = n % a.J3pad;
    for (int x = wave; x < MW * 4; x += NW) {
        acc_t s = red[0][x][lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += red[w][x][lane];
        const int64_t j1 = m0 + (x / 4) * 16 + TR::acc_row(g, x % 4);
        if (j1 < a.J1 && j2 < a.J2 && j3 < a.J3) static_cast<acc_t *>(a.Y)[(j1 * a.J2 + j2) * a.J3 + j3] = s;
    }
}

// Y[j1][j2][j3] = sum_ks Ypart[ks][j1][j2 * J3pad + j3] in increasing ks order.
// Workgroup r owns the row (j1, j2) = (r / J2, r % J2) (one scalar division
// per workgroup instead of three per element), its lanes the j3.
template <typename T>
__global__ void __launch_bounds__(64) k_mode1_reduce(const Mode1Args a) {
    const int64_t row = blockIdx.x;
    const int64_t j1 = row / a.J2, j2 = row - j1 * a.J2;
    const T *Yp = static_cast<const T *>(a.Ypart) + j1 * a.NN + j2 * a.J3pad;
    T *Y = static_cast<T *>(a.Y) + row * a.J3;
    const int64_t ps = a.J1pad * a.NN;
    for (int64_t j3 = threadIdx.x; j3 < a.J3; j3 += 64) {
        const T *p = Yp + j3;
        T s = T(0);
        int k = 0;
        for (; k + 4 <= a.KS; k += 4) {   // four loads in flight, summed in order
            const T v0 = p[k * ps], v1 = p[(k + 1) * ps], v2 = p[(k + 2) * ps], v3 = p[(k + 3) * ps];
            s += v0; s += v1; s += v2; s += v3;
        }
        for (; k < a.KS; ++k) s += p[k * ps];
        Y[j3] = s;
    }
}

// The same sum, 16 bytes per lane: thread t owns four consecutive j3 of row
// t / (J3 / 4) (needs J3 % 4 == 0; J3pad and NN are multiples of 16, so every
// access is 16-byte aligned).  Same order of the terms as k_mode1_reduce.
__global__ void __launch_bounds__(256) k_mode1_reduce4(const Mode1Args a) {
    const int q4 = int(a.J3 / 4);
    const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (t >= a.J1 * a.J2 * q4) return;
    const int64_t row = t / q4, q = t - row * q4;
    const int64_t j1 = row / a.J2, j2 = row - j1 * a.J2;
    const float *p = static_cast<const float *>(a.Ypart) + j1 * a.NN + j2 * a.J3pad + 4 * q;
    const int64_t ps = a.J1pad * a.NN;
    f32x4 s = *reinterpret_cast<const f32x4 *>(p);
    int k = 1;
    for (; k + 4 <= a.KS; k += 4) {   // four loads in flight, summed in order
        const f32x4 v0 = *reinterpret_cast<const f32x4 *>(p + k * ps);
        const f32x4 v1 = *reinterpret_cast<const f32x4 *>(p + (k + 1) * ps);
        const f32x4 v2 = *reinterpret_cast<const f32x4 *>(p + (k + 2) * ps);
        const f32x4 v3 = *reinterpret_cast<const f32x4 *>(p + (k + 3) * ps);
        s += v0; s += v1; s += v2; s += v3;
    }
    for (; k < a.KS; ++k) s += *reinterpret_cast<const f32x4 *>(p + k * ps);
    *reinterpret_cast<f32x4 *>(static_cast<float *>(a.Y) + row * a.J3 + 4 * q) = s;
}

// ---------------------------------------------------------------------------
// Host planning
// ---------------------------------------------------------------------------
// The slab kernel of a call: registers to LDS (k_slab), direct to LDS
// (k_slab_dma), X and C direct to LDS (k_slab_lc).
enum SlabKernel { SLAB_REG, SLAB_DMA, SLAB_LC };

struct ChainPlan {
    int math, xdt;
    SlabKernel kern;
    int WC, NBW, WR, JB, MBK, m1_MW, m1_NW;
    bool m1_small;                // mode 1 by k_mode1_small
    int CB;                       // SLAB_REG: 16-column blocks of a workgroup
    bool rows;                    // SLAB_REG: k_slab_rows in place of k_slab
    int64_t cols;                 // j3 columns per workgroup
    int64_t J3pad, J2pad, J1pad;
    int64_t n_j3_tiles, n_j2_tiles, n_m1_tiles;
    int KS;                       // i1 splits of the mode-1 kernel
    int64_t m1_rows_per_split;
    int S, P;
    int64_t rows_per_split;
    int64_t ldc, ldb, lda;
    size_t fsz;                   // bytes per factor operand element
    size_t acc_sz;
    size_t off_Chi, off_Clo, off_Bhi, off_Blo, off_Ahi, off_Alo, off_V, off_Yp, total;
    bool split;                   // factors need hi/lo
};

static inline size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

static bool combo_ok(int x, int f, int y, int m) {
    if (m == TTM_MATH_F64) return x == TTM_F64 && f == TTM_F64 && y == TTM_F64;
    if (f != TTM_F32 || y != TTM_F32) return false;
    if (m == TTM_MATH_F32 || m == TTM_MATH_BF16 || m == TTM_MATH_BF16X3) return x == TTM_F32 || x == TTM_BF16;
    return false;
}

// V up to here, and few workgroups, go to k_mode1_small (the figures for V are
// there): where the columns alone are many workgroups, k_mode1 needs no split
// either and reads V 256 bytes a row.  Whole chains: 30 x 264 x 32 -> 64, 128, 512
// in float (4096 workgroups) 74.5 us with k_mode1_small, 44.5 with k_mode1; 912 x
// 100 x 30 -> 144, 16, 16 (48) goes to it, 22.7.  Over 725 drawn chains the sides meet at about three workgroups
// of eight waves a compute unit in float and double, two in the bf16 forms.
constexpr int64_t M1_SMALL_V = int64_t(24) << 20;

constexpr int64_t GRID_YZ = 65535;   // workgroups of a launch along y and z

// The direct-to-LDS kernel that takes a shape under the selection `mode`
// (SLAB_REG: none).  Both need 16-byte aligned rows and whole chunks along i3:
// k_slab_dma (256-byte chunks) X already in the operand format, k_slab_lc
// (128-byte chunks) bf16 X with the bf16 forms and four column waves.
// Automatic selection, whole chains measured on both sides (us):
// * k_slab_lc where it applies and the row range of a workgroup holds at least
//   one whole 256-row tile: bf16x3 1024 x 512 x 512 -> 128 231, k_slab 336;
//   512 x 512 x 512 -> 100, 50, 100 110, 140; bf16 1024 x 512 x 512 -> 128 174,
//   197.  (At 64 columns the two are within 7% either way.)
// * k_slab_dma in float past 64 columns (256 x 512 x 512 -> 128: 227, k_slab
//   249; 400 x 500 x 512 -> 100: 408, 462) and, in double, up to 32 where its
//   128-row tiles are full (256 x 256 x 512 -> 16, 30, 12: 58.5, 64.1; -> 16, 30,
//   32: 75.2, 71.4).  The line is drawn for full chips and 100 to 128 columns:
//   up to 96, past 128 and on few workgroups k_slab is ahead there too (float
//   256 x 512 x 512 -> 64, 64, 80 189, 157; 500 x 200 x 512 -> 20, 100, 144 391,
//   270; 64 x 128 x 256 -> 20, 30, 128 30.6, 16.4; double 100 x 128 x 256 -> 16,
//   30, 16 22.9, 16.6).
// * k_slab otherwise: float up to 64 columns (512^3 -> 64: 200, k_slab_dma
//   217; 400 x 300 x 512 -> 64: 115, 133; 400 x 500 x 512 -> 16: 89, 110;
//   256 x 512 x 512 -> 32: 63, 70), double (256^3 -> 64: 70, 82; 128 x 512 x
//   512 -> 100, 120, 128: 255, 452; 64^3 -> 16: 9.0, 11.5), the bf16 forms where
//   k_slab_lc does not apply (512^3 -> 32 bf16x3: 52, 75; bf16 within 4% of each
//   other; but 88 x 336 x 384 -> 24, 6, 72 bf16x3 26.9, 23.5).
static SlabKernel pick_slab(const ttm_shape &s, int xdt, int math, const ChainPlan &p, int mode) {
    const int64_t I3 = s.I[2];
    const bool bf = math == TTM_MATH_BF16 || math == TTM_MATH_BF16X3;
    if (mode == 1 || (I3 * int64_t(dtype_size(xdt))) % 16) return SLAB_REG;
    if (mode == 0 || mode == 3) {
        if (bf && xdt == TTM_BF16 && p.WC == 4 && I3 % 64 == 0 && I3 <= (int64_t(1) << 22) &&
            p.J2pad * round_up(s.I[1], 128) < (int64_t(1) << 30) && (mode == 3 || p.rows_per_split >= LC_TM))
            return SLAB_LC;
        if (mode == 3) return SLAB_REG;
    }
    const bool as_operand = math == TTM_MATH_F64 || (math == TTM_MATH_F32 && xdt == TTM_F32) || (bf && xdt == TTM_BF16);
    if (!as_operand || (I3 * int64_t(dtype_size(xdt))) % 256) return SLAB_REG;
    const int64_t J3 = s.J[2];
    const bool full = s.I[1] % SLAB_TM == 0;
    if (mode == 0 && !(math == TTM_MATH_F32 && J3 > 64) && !(math == TTM_MATH_F64 && J3 <= 32 && full))
        return SLAB_REG;
    return SLAB_DMA;
}

static bool make_plan(const ttm_shape &s, int xdt, int math, int mode, ChainPlan &p) {
    p = ChainPlan();
    p.math = math;
    p.xdt = xdt;
    const int64_t I1 = s.I[0], I2 = s.I[1], I3 = s.I[2];
    const int64_t J1 = s.J[0], J2 = s.J[1], J3 = s.J[2];
    const bool bf = (math == TTM_MATH_BF16 || math == TTM_MATH_BF16X3);
    const int KG = math == TTM_MATH_F64 ? 8 : (math == TTM_MATH_F32 ? 16 : 32);
    const int KC = 2 * KG;
    p.split = (math == TTM_MATH_BF16X3);
    p.fsz = math == TTM_MATH_F64 ? 8 : (bf ? 2 : 4);
    p.acc_sz = math == TTM_MATH_F64 ? 8 : 4;

    // direct-to-LDS kernels: columns (j3) per workgroup and how the 4 waves share them
    const int64_t J3r = round_up(J3, 16), J3b = J3r / 16, jbn = ceil_div(J2, 16);
    if (J3r <= 16) { p.WC = 1; p.NBW = 1; }
    else if (J3r <= 32) { p.WC = 2; p.NBW = 1; }
    else if (J3r <= 64 || math == TTM_MATH_F64) { p.WC = 4; p.NBW = 1; }
    else { p.WC = 4; p.NBW = 2; }
    p.WR = 4 / p.WC;
    p.cols = int64_t(p.WC) * p.NBW * 16;
    int jbmax = math == TTM_MATH_F64 ? 4 : 8;
    auto tile = [&] {
        p.n_j3_tiles = ceil_div(J3r, p.cols);
        p.J3pad = p.n_j3_tiles * p.cols;
        p.JB = jbn > 4 ? jbmax : (jbn > 2 ? 4 : (jbn > 1 ? 2 : 1));   // (past one tile of j2, mode 3 is done again)
        p.n_j2_tiles = ceil_div(jbn, p.JB);
        p.J2pad = p.n_j2_tiles * p.JB * 16;
    };
    tile();
    const int64_t J1b = ceil_div(J1, 16);
    // J within the grids of these tiles and of k_mode1's (where a tiling chosen
    // below is finer, mode 1 keeps k_mode1 and the slab kernel takes another launch)
    if (p.n_j3_tiles > GRID_YZ || p.n_j2_tiles > GRID_YZ || ceil_div(J1b, J1b >= 5 ? 8 : 4) > GRID_YZ) return false;

    // split the i2 rows of a slab so the grid has enough workgroups.  (Five to
    // seven j2 blocks count as two tiles of four, as they were once taken: the
    // splits decide the partials of V, whose order plain bf16 keeps, and their
    // space.)
    const int64_t base = I1 * p.n_j3_tiles * (jbn > 4 && jbn < jbmax ? 2 : p.n_j2_tiles);
    const int64_t max_s = ceil_div(I2, SLAB_TM);
    int64_t S = ceil_div(1024, base);
    if (S < 1) S = 1;
    if (S > max_s) S = max_s;
    if (S > 64) S = 64;
    p.rows_per_split = round_up(ceil_div(I2, S), SLAB_TM);
    p.kern = pick_slab(s, xdt, math, p, mode);
    SlabTile rt = {};
    if (p.kern == SLAB_REG) {
        // all of J3 in one workgroup while two workgroups fit a compute unit
        // (X is read once per j3 tile), in equal tiles past that; in float,
        // bound by its products there, in the tiles that pad least (five blocks
        // are taken as six), each counted as a block more for its reading of X:
        // 143 x 148 x 80 -> 1, 60, 139 in float 42.6 us in two tiles of six, 29.6
        // in three of three
        const bool xf = xdt != TTM_BF16;
        const int most = math == TTM_MATH_F64 || (math == TTM_MATH_BF16X3 && xf) ? 4 : math == TTM_MATH_BF16 ? 8 : 6;
        p.CB = int(ceil_div(J3b, ceil_div(J3b, most)));
        if (p.CB == 5 || p.CB == 7) ++p.CB;
        if (math == TTM_MATH_F32)
            for (int c = 4; c >= 3; --c)
                if (ceil_div(J3b, c) * (c + 1) < ceil_div(J3b, p.CB) * (p.CB + 1)) p.CB = c;
        p.cols = p.CB * 16;
        // j2 tiles of eight blocks; in float and double three of four where two
        // of eight would be a quarter empty and a row is one chunk, which is soon
        // formed again: 40 x 552 x 16 -> 2, 184, 80 in double 56.4 us in two of
        // eight, 40.1 in three of four (longer rows, formed three times: 1.1 to
        // 1.4 times the time)
        jbmax = jbn > 8 && jbn <= 12 && I3 <= KC && !bf ? 4 : 8;
        tile();
        rt = slab_tile(math, xf, p.CB);
        p.WR = rt.WR;
        // k_slab_rows for at most 16 columns j3.  In float and double while J2 is
        // at most 32 (past that k_slab deals the blocks of j2 to its waves: 80 x 8
        // x 96 -> 6, 85, 2 of bf16 in float 9.6 us, here 11.4) and a row at most
        // five chunks (longer rows want two chunks ahead: 800 x 33 x 184 -> 3, 1, 2
        // 19.9 and 22.2).  In plain bf16 while a workgroup has few chunks, or half
        // of its rows and more are past I2 and are not fetched; not for single
        // chunks that fill the chip at most once, nor for long walks: 981 x 8 x 331 -> 32, 2, 1 35.0 and 20.7 us, 896 x
        // 91 x 49 -> 88, 8, 8 21.2 and 19.3, 544 x 248 x 206 -> 48, 6, 14 34.1 and
        // 35.0; past the lines 832 x 869 x 600 -> 1, 1, 8 221 and 240, 53 x 389 x
        // 600 -> 2, 13, 14 of float 20.2 and 23.2, 16 x 22 x 18 -> 2, 1, 1 9.9 and 10.2
        const int64_t nk = ceil_div(I3, KC), walk = ceil_div(std::min(I2, p.rows_per_split), SLAB_TM) * nk;
        p.rows = mode == 0 && J3 <= 16 && !p.split &&
                 (bf ? (walk <= 6 || 2 * I2 <= SLAB_TM) &&
                           (walk > 1 || I1 * ceil_div(I2, p.rows_per_split) * p.n_j2_tiles > 256)
                     : p.JB <= 2 && nk <= 5);
        const int64_t TM = p.rows ? SLAB_TM : rt.TM;
        // row splits: a compute unit's workgroups n take n chunk times where
        // they fill it and about three where one waits out its chunk's trips
        // alone, for as many chunks as a workgroup has and four more for its
        // start and end; and the partials of V are written and read, in units of
        // the bytes of X that a chunk brings every compute unit (not for plain
        // bf16, whose partials are fixed: SlabTile).  (As a share of X's bytes,
        // which on a chip that is not full cost nothing, V kept 16 x 852 x 11 ->
        // 140, 136, 39 in double to one split: 86.6 us, now 32.8.)
        // Counting rounds of workgroups alone (which took one split of 512 x 512 x
        // 500 -> 64 in float, and more than half of a second round idle) gave
        // 242 us there, this 204; 424 x 392 x 48 -> 8 x 15 x 16 in double 40.5 us
        // with its one split, 39.9 with this rule's two.
        const int64_t occ = std::min(4, 163840 / (p.rows ? slab_rows_lds(nk) : rt.lds));
        const double vx = 2.0 * double(I1) * double(p.J2pad) * double(p.J3pad) * double(p.acc_sz) /
                          (256.0 * double(TM * std::min<int64_t>(I3, KC)) * double(dtype_size(xdt)));
        double best = 0;
        const int64_t tiles = ceil_div(I2, TM);
        for (int64_t c = 1; c <= std::min<int64_t>(tiles, 64) && math != TTM_MATH_BF16; c += c < 8 ? 1 : 8) {
            const int64_t per = ceil_div(tiles, c), wg = I1 * p.n_j3_tiles * p.n_j2_tiles * ceil_div(tiles, per);
            const double n = wg > 256 * 8 ? double(wg) / 256 : double(ceil_div(wg, 256));
            const double turns = n > double(8 * occ) ? n / double(occ) : double(ceil_div(int64_t(n + 0.999), occ));
            const double cost = std::max(3.0 * turns, n) * double(per * nk + 4) + vx * double(ceil_div(tiles, per));
            if (c == 1 || cost < best) { best = cost; S = c; p.rows_per_split = per * TM; }
        }
    }

    p.ldc = round_up(I3, KC);
    p.ldb = round_up(I2, SLAB_TM);
    p.lda = round_up(I1, KC);

    ChainPlan first;
    for (bool reduced = false, one_split = false, tight = false;; ) {
        p.S = int(ceil_div(I2, p.rows_per_split));
        p.P = p.S * p.WR;
        // mode-1 kernel: split the i1 range while the column tiles alone leave the
        // GPU short of workgroups (about 512 in all: measured at 1024^3 -> 128^3,
        // fewer, longer splits beat about 1024 once V is prefetched ahead),
        // keeping the partials at most half of V's size
        const int64_t NN = p.J2pad * p.J3pad;
        // mode-1 kernel tiling: MW row blocks and NW column blocks per wave;
        // V of at most SMALL_V bytes goes to the kernel that needs no split
        p.m1_small = I1 * p.P * NN * int64_t(p.acc_sz) <= M1_SMALL_V && ceil_div(J1b, 4) <= GRID_YZ;
        const int64_t small_wg = NN / 16 * ceil_div(J1b, J1b > 2 ? 4 : J1b);
        p.m1_small = p.m1_small && small_wg <= (bf ? 512 : 768);
        // (plain bf16 with four partials and more in each of three and more
        // rounds of the waves, and few rows: 960 x 200 x 16 -> 32, 16, 16 37.0 us
        // with k_mode1_small, 29.1 with k_mode1 over fifteen splits)
        if (math == TTM_MATH_BF16 && p.P >= 4 && I1 > 2 * 8 * KG && J1b <= 2) p.m1_small = false;
        if (p.m1_small) { p.m1_NW = 0; p.m1_MW = J1b > 2 ? 4 : int(J1b); }
        else if (J1b <= 2) { p.m1_NW = 1; p.m1_MW = int(J1b); }
        else { p.m1_NW = 4; p.m1_MW = J1b >= 5 ? 2 : 1; }
        p.MBK = p.m1_NW == 4 ? 4 * p.m1_MW : p.m1_MW;
        p.n_m1_tiles = ceil_div(J1b, p.MBK);
        p.J1pad = p.n_m1_tiles * p.MBK * 16;
        const int64_t wg = (NN / 64) * p.n_m1_tiles;
        int64_t ks = ceil_div(512, wg);
        const int64_t ks_bytes = (I1 * p.P) / (2 * p.J1pad);
        if (ks > ks_bytes) ks = ks_bytes;
        if (ks > ceil_div(I1, KC)) ks = ceil_div(I1, KC);
        if (ks > 64) ks = 64;
        if (ks < 1 || one_split || p.m1_small) ks = 1;
        p.m1_rows_per_split = round_up(ceil_div(I1, ks), KC);
        p.KS = int(ceil_div(I1, p.m1_rows_per_split));

        size_t off = 0;
        auto take = [&](size_t bytes) { size_t o = off; off = al256(off + bytes); return o; };
        // operand arrays (float and double: A is read where it is, and by
        // k_slab B and C too)
        const bool own = bf || p.kern != SLAB_REG;
        p.off_Chi = own ? take(size_t(p.J3pad) * p.ldc * p.fsz) : 0;
        p.off_Clo = p.split ? take(size_t(p.J3pad) * p.ldc * p.fsz) : 0;
        p.off_Bhi = own ? take(size_t(p.J2pad) * p.ldb * p.fsz) : 0;
        p.off_Blo = p.split ? take(size_t(p.J2pad) * p.ldb * p.fsz) : 0;
        p.off_Ahi = bf ? take(size_t(p.J1pad) * p.lda * p.fsz) : 0;
        p.off_Alo = p.split ? take(size_t(p.J1pad) * p.lda * p.fsz) : 0;
        p.off_V = take(size_t(I1) * p.P * p.J2pad * p.J3pad * p.acc_sz);
        p.off_Yp = p.KS > 1 ? take(size_t(p.KS) * p.J1pad * p.J2pad * p.J3pad * p.acc_sz) : 0;
        p.total = off;
        // the library-owned scratch holds what it holds with one row split, one
        // mode-1 split and tiles of at most 64 rows j2 and 64 columns j3 (which
        // pad J2 and J3 least): splits and tiles that pass it are taken back,
        // unless even those do (ttm_chain then loses by fewer: bf16x3 1024 x 512 x
        // 771 -> 128 897 us with one split and small tiles, 525 as first planned)
        if (p.kern != SLAB_REG || math == TTM_MATH_BF16 || p.total <= TTM_NOALLOC_SCRATCH_BYTES) break;
        if (!reduced) {
            first = p;
            reduced = true;
        }
        if (p.S > 1) {
            p.rows_per_split = round_up(ceil_div(I2, p.S - 1), p.rows ? SLAB_TM : rt.TM);
        } else if (!one_split && p.KS > 1) {
            one_split = true;
        } else if (!tight) {
            tight = true;
            p.CB = int(ceil_div(J3b, ceil_div(J3b, 4)));
            p.cols = p.CB * 16;
            jbmax = 4;
            tile();
            rt = slab_tile(math, xdt != TTM_BF16, p.CB);
            p.rows_per_split = round_up(I2, p.rows ? SLAB_TM : rt.TM);
        } else {
            p = first;
            break;
        }
    }
    // launch-grid limits
    return I1 * p.S <= 0x7fffffffLL && p.n_j2_tiles <= GRID_YZ && p.J2pad * p.J3pad / 64 <= 0x7fffffffLL && J1 * J2 <= 0x7fffffffLL;
}

template <int MATH, typename XT, int CB, int JB>
static int launch_slab(const ChainPlan &p, const SlabArgs &a, hipStream_t st) {
    typedef SlabCfg<MATH, XT, CB> CF;
    typedef typename CF::TR::fac_t FT;
    typedef typename CF::TR::acc_t acc_t;
    static std::atomic<uint64_t> attr_set{0};
    if (int rc = ensure_lds_limit(reinterpret_cast<const void *>(&k_slab<MATH, XT, CB, JB>), CF::LDS, attr_set))
        return rc;
    // (more than one launch only for J3 in the millions)
    for (int64_t t = 0; t < p.n_j3_tiles; t += GRID_YZ) {
        SlabArgs b = a;
        const int64_t col = t * CB * 16, coff = col * (MATH == M_F32 || MATH == M_F64 ? a.I3 : a.ldc);
        b.Chi = static_cast<const FT *>(a.Chi) + coff;
        b.Clo = a.Clo ? static_cast<const FT *>(a.Clo) + coff : nullptr;
        b.V = static_cast<acc_t *>(a.V) + col;
        b.J3 = a.J3 - col;
        dim3 grid(unsigned(a.I1 * a.S), unsigned(std::min(p.n_j3_tiles - t, GRID_YZ)), unsigned(p.n_j2_tiles));
        const int rc = launch("ttm_slab", st, [&] {
            hipLaunchKernelGGL((k_slab<MATH, XT, CB, JB>), grid, dim3(SLAB_THREADS), CF::LDS, st, b);
        });
        if (rc) return rc;
    }
    return TTM_OK;
}

template <int MATH, typename XT, int CB>
static int dispatch_slab_reg_jb(const ChainPlan &p, const SlabArgs &a, hipStream_t st) {
    switch (p.JB) {
        case 1: return launch_slab<MATH, XT, CB, 1>(p, a, st);
        case 2: return launch_slab<MATH, XT, CB, 2>(p, a, st);
        case 4: return launch_slab<MATH, XT, CB, 4>(p, a, st);
        default: return launch_slab<MATH, XT, CB, 8>(p, a, st);
    }
}

template <int MATH, typename XT>
static int dispatch_slab_rows(const ChainPlan &p, const SlabArgs &a, hipStream_t st) {
    const dim3 grid(unsigned(a.I1 * a.S), 1, unsigned(p.n_j2_tiles));
    const int lds = slab_rows_lds(MATH == M_BF16 ? 0 : ceil_div(a.I3, 2 * MathTraits<MATH>::KG));
    return launch("ttm_slab", st, [&] {
        auto go = [&](auto k) { hipLaunchKernelGGL(k, grid, dim3(SLAB_THREADS), lds, st, a); };
        if (p.JB == 1) return go(k_slab_rows<MATH, XT, 1>);
        if (p.JB == 2) return go(k_slab_rows<MATH, XT, 2>);
        if constexpr (MATH == M_BF16) {
            if (p.JB == 4) return go(k_slab_rows<MATH, XT, 4>);
            return go(k_slab_rows<MATH, XT, 8>);
        }
    });
}

template <int MATH, typename XT>
static int dispatch_slab_reg(const ChainPlan &p, const SlabArgs &a, hipStream_t st) {
    if constexpr (MATH != M_BF16X3) if (p.rows) return dispatch_slab_rows<MATH, XT>(p, a, st);
    switch (p.CB) {
        case 1: return dispatch_slab_reg_jb<MATH, XT, 1>(p, a, st);
        case 2: return dispatch_slab_reg_jb<MATH, XT, 2>(p, a, st);
        case 3: return dispatch_slab_reg_jb<MATH, XT, 3>(p, a, st);
        case 4: return dispatch_slab_reg_jb<MATH, XT, 4>(p, a, st);
        case 6:
            if constexpr (MATH == M_F32 || MATH == M_BF16 || (MATH == M_BF16X3 && !SlabCfg<MATH, XT, 6>::XLO))
                return dispatch_slab_reg_jb<MATH, XT, 6>(p, a, st);
            return TTM_ERR_UNSUPPORTED;
        case 8:
            if constexpr (MATH == M_BF16) return dispatch_slab_reg_jb<MATH, XT, 8>(p, a, st);
            return TTM_ERR_UNSUPPORTED;
        default: return TTM_ERR_UNSUPPORTED;
    }
}

template <int MATH, typename XT, int WC, int NBW, int JB>
static int launch_slab_direct(const ChainPlan &p, const SlabArgs &a, hipStream_t st) {
    typedef typename MathTraits<MATH>::lds_t LT;
    dim3 grid(unsigned(a.I1 * a.S), unsigned(p.n_j3_tiles), unsigned(p.n_j2_tiles));
    if constexpr (std::is_same<XT, LT>::value) {
        if (p.kern == SLAB_DMA)
            return launch("ttm_slab", st, [&] {
                hipLaunchKernelGGL((k_slab_dma<MATH, WC, NBW, JB>), grid, dim3(SLAB_THREADS), 0, st, a);
            });
    }
    if constexpr (WC == 4 && (MATH == M_BF16 || MATH == M_BF16X3) && std::is_same<XT, uint16_t>::value) {
        if (p.kern == SLAB_LC)
            return launch("ttm_slab", st, [&] {
                hipLaunchKernelGGL((k_slab_lc<MATH, NBW, JB>), grid, dim3(LC_THREADS), 0, st, a);
            });
    }
    return TTM_ERR_UNSUPPORTED;
}

template <int MATH, typename XT, int WC, int NBW>
static int dispatch_slab_jb(const ChainPlan &p, const SlabArgs &a, hipStream_t st) {
    switch (p.JB) {
        case 1: return launch_slab_direct<MATH, XT, WC, NBW, 1>(p, a, st);
        case 2: return launch_slab_direct<MATH, XT, WC, NBW, 2>(p, a, st);
        case 4: return launch_slab_direct<MATH, XT, WC, NBW, 4>(p, a, st);
        default:
            if constexpr (MATH != M_F64) return launch_slab_direct<MATH, XT, WC, NBW, 8>(p, a, st);
            return TTM_ERR_UNSUPPORTED;
    }
}

template <int MATH, typename XT>
static int dispatch_slab(const ChainPlan &p, const SlabArgs &a, hipStream_t st) {
    if (p.kern == SLAB_REG) return dispatch_slab_reg<MATH, XT>(p, a, st);
    if (p.WC == 1) return dispatch_slab_jb<MATH, XT, 1, 1>(p, a, st);
    if (p.WC == 2) return dispatch_slab_jb<MATH, XT, 2, 1>(p, a, st);
    if (p.NBW == 1) return dispatch_slab_jb<MATH, XT, 4, 1>(p, a, st);
    if constexpr (MATH != M_F64) return dispatch_slab_jb<MATH, XT, 4, 2>(p, a, st);
    return TTM_ERR_UNSUPPORTED;
}

template <int MATH>
static int dispatch_mode1(const ChainPlan &p, const Mode1Args &a, hipStream_t st) {
    typedef typename MathTraits<MATH>::acc_t acc_t;
    if (p.m1_small) {
        dim3 grid(unsigned(p.J2pad * p.J3pad / 16), 1, unsigned(p.n_m1_tiles));
        // sixteen waves where eight would leave most of the chip idle (not in
        // the bf16 forms, whose eight values a lane spill there: 389 x 232 x 136
        // -> 6 x 15 x 8 17.7 us, eight waves 9.2; double 424 x 392 x 48 -> 8 x
        // 15 x 16 5.4 us, eight waves 7.6)
        return launch("ttm_mode1", st, [&] {
            auto go = [&](auto k, int nw) { hipLaunchKernelGGL(k, grid, dim3(64 * nw), 0, st, a); };
            if constexpr (MATH == M_F32 || MATH == M_F64)
                if (grid.x * grid.z < 256 && p.m1_MW <= 2)
                    return p.m1_MW == 1 ? go(k_mode1_small<MATH, 1, 16>, 16) : go(k_mode1_small<MATH, 2, 16>, 16);
            if (p.m1_MW == 1) go(k_mode1_small<MATH, 1, 8>, 8);
            else if (p.m1_MW == 2) go(k_mode1_small<MATH, 2, 8>, 8);
            else go(k_mode1_small<MATH, 4, 8>, 8);
        });
    }
    dim3 grid(unsigned(p.J2pad * p.J3pad / 64), unsigned(p.KS), unsigned(p.n_m1_tiles));
    auto go = [&](auto kern) {
        return launch("ttm_mode1", st, [&] { hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, a); });
    };
    int rc;
    if (p.m1_NW == 1) rc = p.m1_MW == 1 ? go(k_mode1<MATH, 1, 1>) : go(k_mode1<MATH, 2, 1>);
    else rc = p.m1_MW == 1 ? go(k_mode1<MATH, 1, 4>) : go(k_mode1<MATH, 2, 4>);
    if (rc || p.KS == 1) return rc;
    if (MATH != M_F64 && a.J3 % 4 == 0 && aligned(a.Y, 16)) {
        const int64_t n4 = a.J1 * a.J2 * (a.J3 / 4);
        return launch("ttm_mode1_reduce", st, [&] {
            hipLaunchKernelGGL(k_mode1_reduce4, dim3(unsigned(ceil_div(n4, 256))), dim3(256), 0, st, a);
        });
    }
    return launch("ttm_mode1_reduce", st, [&] {
        hipLaunchKernelGGL((k_mode1_reduce<acc_t>), dim3(unsigned(a.J1 * a.J2)), dim3(64), 0, st, a);
    });
}

template <int MATH>
static int run_chain(const ChainPlan &p, const ttm_shape &s, const void *X, const void *A, const void *B,
                     const void *C, void *Y, unsigned char *ws, hipStream_t st) {
    // 1. factor operands
    PrepArgs pa;
    const void *src[3] = {A, B, C};
    const size_t offh[3] = {p.off_Ahi, p.off_Bhi, p.off_Chi}, offl[3] = {p.off_Alo, p.off_Blo, p.off_Clo};
    const int64_t Jpad[3] = {p.J1pad, p.J2pad, p.J3pad}, ld[3] = {p.lda, p.ldb, p.ldc};
    int64_t maxn = 0;
    for (int f = 0; f < 3; ++f) {
        pa.src[f] = src[f];
        pa.hi[f] = ws + offh[f];
        pa.lo[f] = p.split ? ws + offl[f] : nullptr;
        pa.J[f] = s.J[f];
        pa.I[f] = s.I[f];
        pa.Jpad[f] = Jpad[f];
        pa.ld[f] = ld[f];
        pa.perm32[f] = (f == 1 && (MATH == M_BF16 || MATH == M_BF16X3)) ? 1 : 0;
        maxn = std::max<int64_t>(maxn, Jpad[f] * ld[f]);
    }
    // float and double: the register-staged kernel and mode 1 read the factors
    // where they are; the direct-to-LDS kernel does where the padded arrays
    // would equal them (rows a multiple of the tile, row length a multiple of
    // the k chunk), and else has B and C prepared
    const void *fac[3];
    for (int f = 0; f < 3; ++f) fac[f] = ws + offh[f];
    bool prepare = true;
    if constexpr (MATH == M_F32 || MATH == M_F64) {
        fac[0] = A;
        pa.Jpad[0] = 0;
        bool direct = true;
        for (int f = 1; f < 3; ++f) direct = direct && Jpad[f] == s.J[f] && ld[f] == s.I[f] && aligned(src[f], 16);
        prepare = p.kern != SLAB_REG && !direct;
        if (!prepare) { fac[1] = B; fac[2] = C; }
    }
    dim3 pgrid(unsigned(std::min<int64_t>(ceil_div(maxn, 256), 4096)), 3);
    int rc = TTM_OK;
    if (prepare) {
        if constexpr (MATH == M_F64)
            rc = launch("ttm_prep", st,
                        [&] { hipLaunchKernelGGL((k_prep_factors<double, MATH>), pgrid, dim3(256), 0, st, pa); });
        else
            rc = launch("ttm_prep", st,
                        [&] { hipLaunchKernelGGL((k_prep_factors<float, MATH>), pgrid, dim3(256), 0, st, pa); });
    }
    if (rc) return rc;

    // 2. slab kernel (modes 3 and 2)
    SlabArgs sa;
    sa.X = X;
    sa.I1 = s.I[0]; sa.I2 = s.I[1]; sa.I3 = s.I[2];
    sa.Chi = fac[2]; sa.Clo = p.split ? ws + p.off_Clo : nullptr; sa.ldc = p.ldc;
    sa.Bhi = fac[1]; sa.Blo = p.split ? ws + p.off_Blo : nullptr; sa.ldb = p.ldb;
    sa.J2 = s.J[1]; sa.J3 = s.J[2];
    sa.V = ws + p.off_V;
    sa.J2pad = p.J2pad; sa.J3pad = p.J3pad;
    sa.P = p.P; sa.S = p.S;
    sa.rows_per_split = p.rows_per_split;
    if constexpr (MATH == M_F64) rc = dispatch_slab<M_F64, double>(p, sa, st);
    else if (p.xdt == TTM_BF16) rc = dispatch_slab<MATH, uint16_t>(p, sa, st);
    else rc = dispatch_slab<MATH, float>(p, sa, st);
    if (rc) return rc;

    // 3. mode 1
    Mode1Args ma;
    ma.Ahi = fac[0]; ma.Alo = p.split ? ws + p.off_Alo : nullptr; ma.lda = MATH == M_F32 || MATH == M_F64 ? s.I[0] : p.lda;
    ma.V = ws + p.off_V; ma.I1 = s.I[0]; ma.P = p.P;
    ma.NN = p.J2pad * p.J3pad; ma.J3pad = p.J3pad;
    ma.Y = Y; ma.Ypart = p.KS > 1 ? ws + p.off_Yp : nullptr;
    ma.J1 = s.J[0]; ma.J2 = s.J[1]; ma.J3 = s.J[2]; ma.J1pad = p.J1pad;
    ma.KS = p.KS; ma.rows_per_split = p.m1_rows_per_split;
    return dispatch_mode1<MATH>(p, ma, st);
}

static int validate_shape(const ttm_shape *s) {
    if (!s) return TTM_ERR_INVALID_ARG;
    for (int n = 0; n < 3; ++n)
        if (s->I[n] < 1 || s->J[n] < 1 || s->I[n] > (int64_t(1) << 31) || s->J[n] > (int64_t(1) << 31))
            return TTM_ERR_INVALID_ARG;
    if (checked_prod(checked_prod(s->I[0], s->I[1]), s->I[2]) < 0) return TTM_ERR_INVALID_ARG;
    if (checked_prod(checked_prod(s->J[0], s->J[1]), s->J[2]) < 0) return TTM_ERR_INVALID_ARG;
    return TTM_OK;
}

// Argument checks shared by the entry points of the chain (everything but
// the workspace) and the plan for the shape.
static int chain_check(const ttm_shape *s, const void *X, int x_dtype, const void *A, const void *B,
                       const void *C, int f_dtype, const void *Y, int y_dtype, int math, ChainPlan &p) {
    int rc = validate_shape(s);
    if (rc) return rc;
    if (!combo_ok(x_dtype, f_dtype, y_dtype, math)) return TTM_ERR_UNSUPPORTED;
    if (!X || !A || !B || !C || !Y) return TTM_ERR_INVALID_ARG;
    const size_t fs = dtype_size(f_dtype), ys = dtype_size(y_dtype), xs = dtype_size(x_dtype);
    if (!aligned(X, 16) || !aligned(Y, 16) || !aligned(A, fs) || !aligned(B, fs) || !aligned(C, fs))
        return TTM_ERR_INVALID_ARG;
    if (!make_plan(*s, x_dtype, math, slab_kernel_mode(), p)) return TTM_ERR_UNSUPPORTED;
    const size_t ny = size_t(s->J[0] * s->J[1] * s->J[2]) * ys;
    const size_t nx = size_t(s->I[0] * s->I[1] * s->I[2]) * xs;
    if (overlaps(Y, ny, X, nx) || overlaps(Y, ny, A, size_t(s->J[0] * s->I[0]) * fs) ||
        overlaps(Y, ny, B, size_t(s->J[1] * s->I[1]) * fs) || overlaps(Y, ny, C, size_t(s->J[2] * s->I[2]) * fs))
        return TTM_ERR_ALIAS;
    return TTM_OK;
}

// Workspace checks and the launches.
static int chain_run(const ChainPlan &p, const ttm_shape *s, const void *X, const void *A, const void *B,
                     const void *C, void *Y, int math, void *ws, size_t ws_bytes, hipStream_t st) {
    if (!ws || ws_bytes < p.total) return TTM_ERR_WORKSPACE;
    if (!aligned(ws, 16)) return TTM_ERR_INVALID_ARG;
    const size_t fs = p.math == TTM_MATH_F64 ? 8 : 4, ys = fs, xs = dtype_size(p.xdt);
    const size_t ny = size_t(s->J[0] * s->J[1] * s->J[2]) * ys;
    const size_t nx = size_t(s->I[0] * s->I[1] * s->I[2]) * xs;
    if (overlaps(Y, ny, ws, p.total) || overlaps(ws, p.total, X, nx) ||
        overlaps(ws, p.total, A, size_t(s->J[0] * s->I[0]) * fs) ||
        overlaps(ws, p.total, B, size_t(s->J[1] * s->I[1]) * fs) ||
        overlaps(ws, p.total, C, size_t(s->J[2] * s->I[2]) * fs))
        return TTM_ERR_ALIAS;
    unsigned char *w = static_cast<unsigned char *>(ws);
    switch (math) {
        case TTM_MATH_F64: return run_chain<M_F64>(p, *s, X, A, B, C, Y, w, st);
        case TTM_MATH_F32: return run_chain<M_F32>(p, *s, X, A, B, C, Y, w, st);
        case TTM_MATH_BF16: return run_chain<M_BF16>(p, *s, X, A, B, C, Y, w, st);
        case TTM_MATH_BF16X3: return run_chain<M_BF16X3>(p, *s, X, A, B, C, Y, w, st);
        default: return TTM_ERR_UNSUPPORTED;
    }
}

// ---------------------------------------------------------------------------
// Library-owned scratch for ttm_chain_noalloc: a fixed device array in this
// code object, one copy per GPU, held until the process ends.  Host code
// never uses the array's name as an address (on the host it names a
// stand-in); the device address comes from hipGetSymbolAddress, taken once
// per device with that device current and kept per device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[TTM_NOALLOC_SCRATCH_BYTES];

static std::mutex g_scratch_mu;
static void *g_scratch_ptr[64];

static int noalloc_scratch(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return TTM_ERR_HIP;
    if (dev < 0 || dev >= 64) return TTM_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return TTM_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return TTM_OK;
}

}  // namespace ttm

using namespace ttm;

extern "C" {

int ttm_chain_supported(int x, int f, int y, int m) { return combo_ok(x, f, y, m) ? 1 : 0; }

size_t ttm_chain_workspace_size(const ttm_shape *s, int x_dtype, int math) {
    if (validate_shape(s) != TTM_OK) return 0;
    const int f = math == TTM_MATH_F64 ? TTM_F64 : TTM_F32;
    if (!combo_ok(x_dtype, f, f, math)) return 0;
    // enough for every kernel selection, which may change between the query
    // and the call: the register-staged kernel's plan, k_slab_rows' (its row
    // splits are its own) and the direct ones' (which share theirs)
    ChainPlan p, d;
    if (!make_plan(*s, x_dtype, math, 1, p)) return 0;
    size_t total = p.total;
    if (make_plan(*s, x_dtype, math, 0, d)) total = std::max(total, d.total);
    for (int mode : {2, 3})
        if (make_plan(*s, x_dtype, math, mode, d) && d.kern != SLAB_REG) return std::max(total, d.total);
    return total;
}

int ttm_chain(const ttm_shape *s, const void *X, int x_dtype, const void *A, const void *B, const void *C,
              int f_dtype, void *Y, int y_dtype, int math, void *ws, size_t ws_bytes, void *stream) {
    ChainPlan p;
    int rc = chain_check(s, X, x_dtype, A, B, C, f_dtype, Y, y_dtype, math, p);
    if (rc) return rc;
    return chain_run(p, s, X, A, B, C, Y, math, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

int ttm_chain_noalloc(const ttm_shape *s, const void *X, int x_dtype, const void *A, const void *B,
                      const void *C, int f_dtype, void *Y, int y_dtype, int math, void *stream) {
    ChainPlan p;
    int rc = chain_check(s, X, x_dtype, A, B, C, f_dtype, Y, y_dtype, math, p);
    if (rc) return rc;
    if (p.total > TTM_NOALLOC_SCRATCH_BYTES) return TTM_ERR_WORKSPACE;
    void *ws = nullptr;
    rc = noalloc_scratch(&ws);
    if (rc) return rc;
    return chain_run(p, s, X, A, B, C, Y, math, ws, TTM_NOALLOC_SCRATCH_BYTES, static_cast<hipStream_t>(stream));
}

}  // extern "C"
