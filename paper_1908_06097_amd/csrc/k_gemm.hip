// Legendre transforms as grouped, even/odd-split GEMMs on the CDNA4 matrix
// cores, one launch per direction covering every wavenumber m.
//
// For each m the n-range splits by the parity p of n - m, and the equatorial
// symmetry P̄_n^m(-mu) = (-1)^(n-m) P̄_n^m(mu) lets one product over the
// northern rings serve both hemispheres:
//
//   inverse:  S_p[r][c] = sum_k P_p[r][k] B_p[k][c],   B_p[k][c] = a^m_{m+p+2k}
//             F_m(north r) = S_0 + S_1,  F_m(south r) = S_0 - S_1
//   direct:   D_p[k][c] = sum_r P_p[r][k] A_p[r][c],
//             A_p[r][c] = q_r (G_m(north r) + (-1)^p G_m(south r))
//
// with c running over (field, re/im) pairs (the table is real), r over the
// R_m northern rings carrying m and q_r = w_r / 2 (direct transform) or 1
// (adjoint of the inverse).  The spectral operand is read from / written to
// the caller's [field][nspec] array directly (the pack and unpack steps are
// fused into the tile loads and the epilogue), and the Fourier operand lives
// in the [ring][m][field] workspace that the ring FFTs read and write.
//
// The paper treats this step only as part of the SH dwarf (Section 3.1.1);
// the design (grouped launch, XCD-aware work lists, LDS-staged tiles, MFMA)
// is this library's own.
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "shtx_internal.h"

namespace shtx {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Acc;
template <>
struct Acc<float> {
    typedef f32x4 type;
};
template <>
struct Acc<double> {
    typedef f64x4 type;
};

// 16x16x4 MFMA: lane l supplies A[l%16][l/16] and B[l/16][l%16].  It holds
// D[i][l%16] for v = 0..3 with i = 4(l/16) + v for the FP32 form and
// i = l/16 + 4v for the FP64 form (the two differ on CDNA).
__device__ inline f32x4 mfma16x16x4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ inline f64x4 mfma16x16x4(double a, double b, f64x4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <typename T>
__device__ inline int acc_row(int lane, int v)
{
    return sizeof(T) == 8 ? (lane >> 4) + 4 * v : 4 * (lane >> 4) + v;
}

struct GemmArgs {
    const void *tab;  // table for the A operand
    const MBlock *mb;
    const GemmItem *items;
    const RingPair *ring_pair;  // per northern ring: Fourier offsets of it and its mirror
    const void *ring_q;         // per northern ring: w_j / 2 (grid precision)
    const void *in;
    void *out;
    int trunc, nlat, nfld;
    int adjoint;
    int64_t nspec;
    // split IEEE-half form: per-field largest magnitude of the data source
    // (float bits) and the factor that turns it into a bound on the data
    // operand's entries
    const unsigned *fmax;
    float dbound;
};

__device__ inline int64_t spec_base(int trunc, int m) { return (int64_t)m * (2 * trunc + 3 - m) / 2; }

// ---------------------------------------------------------------------------
// FP64.  NW (4 or 8) waves as 2 x (NW/2), each owning a (BM/2) x
// (2 BN/NW) tile per parity.  LDS tiles are K-major (As[buf][p][kappa][i],
// Bs[buf][p][kappa][j]) and double-buffered: the global loads of stage s+1
// are issued into registers before the MFMAs of stage s and written to the
// other buffer after them, with one barrier per stage.
//
// INV: rows i = northern rings of the m band, kappa = k, A = table [p][k][r],
//      B = spectral coefficients read straight from spec[f][index(m, n)].
// DIR: rows i = k, kappa = rings, A = table [p][r][k], B = hemispheric
//      fold of the Fourier workspace q_r (G_north +- G_south).
// ---------------------------------------------------------------------------
template <typename T>
struct __attribute__((aligned(2 * sizeof(T)))) Vec2 {
    T x, y;
};

template <typename T, int BM, int BN, int BK, bool INV, int NW = 4>
__global__ __launch_bounds__(64 * NW, 2) void k_leg_mfma(GemmArgs a)
{
    // NW waves as 2 x (NW / 2): rows split in two, columns in NW / 2
    constexpr int NT = 64 * NW, NWN = NW / 2;
    constexpr int WM = BM / 2, WN = BN / NWN, FM = WM / 16, FN = WN / 16;
    static_assert(NW == 4 || NW == 8, "4 or 8 waves per block");
    constexpr int LDA = BM + 16, LDB = BN + 16;
    constexpr int VEC = 16 / sizeof(T);                 // elements per 16-byte table load
    constexpr int NA = (2 * BK * BM) / (VEC * NT);      // table loads per thread per stage
    // complex operand loads per thread per stage: INV reads BN/2 fields x 2 BK
    // coefficients, DIR reads BK rings x BN/2 fields (north and south each)
    constexpr int NB = INV ? (BK * BN) / NT : (BK * BN) / (2 * NT);
    constexpr int NM = INV ? 1 : NB;  // ring metadata per thread (DIR)
    static_assert(NA * VEC * NT == 2 * BK * BM, "table tile must split evenly");
    static_assert(NB * (INV ? NT : 2 * NT) == BK * BN, "operand tile must split evenly");
    static_assert(BK == 16 && BN >= 32, "operand swizzle assumes 16-deep stages");
    typedef typename Acc<T>::type V;
    typedef T VecT __attribute__((ext_vector_type(VEC)));
    // operand tiles As[buf][p][kappa][i], Bs[buf][p][kappa][j]; the direct
    // GEMM reuses the same LDS to stage its output tile
    constexpr int NSMEM = 2 * 2 * BK * (LDA + LDB);
    __shared__ __attribute__((aligned(16))) T smem[NSMEM];
    auto As = reinterpret_cast<T(*)[2][BK][LDA]>(smem);
    auto Bs = reinterpret_cast<T(*)[2][BK][LDB]>(smem + 2 * 2 * BK * LDA);

    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const GemmItem it = a.items[item];
    if (it.m < 0) return;
    const int m = it.m;
    const MBlock b = a.mb[m];
    const int row0 = it.tr * BM, col0 = it.tc * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = (wave / NWN) * WM, wc = (wave % NWN) * WN;
    const int ncol = 2 * a.nfld;
    const int64_t pstride = (int64_t)b.Kp * b.Rp;
    const T *A0 = (const T *)a.tab + b.off;
    const int lda_g = INV ? b.Rp : b.Kp;  // global row stride of the table tile
    const int64_t sb = spec_base(a.trunc, m);
    const int kend = INV ? b.K0 : b.R;
    const int nstages = (kend + BK - 1) / BK;

    // INV stores the coefficient tile with the field index XOR-swizzled by
    // its (parity, k) slot, so that the column-strided stores of one wave
    // hit distinct LDS banks; the MFMA reads undo the swizzle.
    auto bswz = [](int p, int q) { return 2 * (((q >> 1) & 3) | (p << 2)); };

    VecT ra[NA];
    Vec2<T> rb0[NB], rb1[NB];
    // DIR: Fourier offsets and weights of each thread's rings, fetched one
    // stage ahead of the data so that no data load waits on them
    RingPair mp1[NM], mp2[NM];
    T mq1[NM], mq2[NM];

    auto meta = [&](int kk, RingPair *mp, T *mq) {
#pragma unroll
        for (int v = 0; v < NM; ++v) {
            int r = kk + (tid + v * NT) / (BN / 2);
            RingPair o = {-1, -1};
            T w = T(0);
            if (r < b.R) {
                o = a.ring_pair[b.j0 + r];
                w = a.adjoint ? T(1) : ((const T *)a.ring_q)[b.j0 + r];
            }
            mp[v] = o;
            mq[v] = w;
        }
    };
    // global -> registers (no arithmetic on the loaded values here, so that
    // nothing waits for the loads before the MFMAs of the current stage)
    auto load = [&](int kk) {
#pragma unroll
        for (int v = 0; v < NA; ++v) {
            int idx = tid + v * NT;
            int p = idx / (BK * BM / VEC), rem = idx - p * (BK * BM / VEC);
            int q = rem / (BM / VEC), i = (rem - q * (BM / VEC)) * VEC;
            ra[v] = *reinterpret_cast<const VecT *>(A0 + p * pstride + (int64_t)(kk + q) * lda_g + row0 + i);
        }
        if (INV) {
            const Vec2<T> *spec = (const Vec2<T> *)a.in;
#pragma unroll
            for (int v = 0; v < NB; ++v) {
                int idx = tid + v * NT;
                int fl = idx / (2 * BK), t = idx - fl * (2 * BK);
                int f = col0 / 2 + fl, nrel = 2 * kk + t;
                Vec2<T> z = {T(0), T(0)};
                if (f < a.nfld && m + nrel <= a.trunc) z = spec[(int64_t)f * a.nspec + sb + nrel];
                rb0[v] = z;
            }
        } else {
            const Vec2<T> *four = (const Vec2<T> *)a.in;
#pragma unroll
            for (int v = 0; v < NB; ++v) {
                int idx = tid + v * NT;
                int cp = idx % (BN / 2);
                int f = col0 / 2 + cp;
                Vec2<T> gn = {T(0), T(0)}, gs = {T(0), T(0)};
                if (mp1[v].n >= 0 && f < a.nfld) {
                    gn = four[((int64_t)mp1[v].n + m) * a.nfld + f];
                    gs = four[((int64_t)mp1[v].s + m) * a.nfld + f];
                }
                rb0[v] = gn;
                rb1[v] = gs;
            }
        }
    };
    // registers -> LDS: INV zeroes Im a^0_n, DIR folds the hemispheres
    auto store = [&](int buf) {
#pragma unroll
        for (int v = 0; v < NA; ++v) {
            int idx = tid + v * NT;
            int p = idx / (BK * BM / VEC), rem = idx - p * (BK * BM / VEC);
            int q = rem / (BM / VEC), i = (rem - q * (BM / VEC)) * VEC;
            *reinterpret_cast<VecT *>(&As[buf][p][q][i]) = ra[v];
        }
        if (INV) {
#pragma unroll
            for (int v = 0; v < NB; ++v) {
                int idx = tid + v * NT;
                int fl = idx / (2 * BK), t = idx - fl * (2 * BK);
                int p = t & 1, q = t >> 1;
                Vec2<T> z = rb0[v];
                if (m == 0) z.y = T(0);
                *reinterpret_cast<Vec2<T> *>(&Bs[buf][p][q][(2 * fl) ^ bswz(p, q)]) = z;
            }
        } else {
#pragma unroll
            for (int v = 0; v < NB; ++v) {
                int idx = tid + v * NT;
                int q = idx / (BN / 2), cp = idx - q * (BN / 2);
                const T w = mq1[v];
                const Vec2<T> gn = rb0[v], gs = rb1[v];
                Vec2<T> s0 = {w * (gn.x + gs.x), w * (gn.y + gs.y)};
                Vec2<T> s1 = {w * (gn.x - gs.x), w * (gn.y - gs.y)};
                *reinterpret_cast<Vec2<T> *>(&Bs[buf][0][q][2 * cp]) = s0;
                *reinterpret_cast<Vec2<T> *>(&Bs[buf][1][q][2 * cp]) = s1;
            }
        }
    };

    V acc[2][FM][FN];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[p][i][j] = V{};

    // per-lane column of the B reads for each k step and parity (INV swizzle)
    int bcol[BK / 4][2];
#pragma unroll
    for (int q = 0; q < BK; q += 4)
#pragma unroll
        for (int p = 0; p < 2; ++p)
            bcol[q / 4][p] = INV ? ((lane & 15) ^ bswz(p, q + (lane >> 4))) : (lane & 15);

    if (!INV) meta(0, mp1, mq1);
    load(0);
    store(0);
    if (!INV && nstages > 1) meta(BK, mp1, mq1);
    __syncthreads();
    // Row fragments of this wave's sub-tile that hold data: on the ragged
    // edge of an m block the fragments past the last valid row (and a wave
    // wholly past the valid rows or columns) skip their LDS reads and MFMAs,
    // still loading and storing their share of the operand tiles.  The K
    // loop is instantiated per count so that the accumulators stay in place.
    const int nfa = __builtin_amdgcn_readfirstlane(
        col0 + wc < ncol ? min(FM, max(0, ((INV ? b.R : b.K0) - row0 - wr + 15) / 16)) : 0);
    auto kloop = [&](auto nfa_c) __attribute__((always_inline)) {
        constexpr int NFA = decltype(nfa_c)::value;
        for (int s = 0; s < nstages; ++s) {
            const int cur = s & 1;
            const bool more = s + 1 < nstages;
            if (more) load((s + 1) * BK);
            if (!INV && s + 2 < nstages) meta((s + 2) * BK, mp2, mq2);
            if constexpr (NFA > 0) {
#pragma unroll
                for (int q = 0; q < BK; q += 4) {
                    const int qq = q + (lane >> 4);
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        T av[NFA], bv[FN];
#pragma unroll
                        for (int i = 0; i < NFA; ++i) av[i] = As[cur][p][qq][wr + i * 16 + (lane & 15)];
#pragma unroll
                        for (int j = 0; j < FN; ++j) bv[j] = Bs[cur][p][qq][wc + j * 16 + bcol[q / 4][p]];
#pragma unroll
                        for (int i = 0; i < NFA; ++i)
#pragma unroll
                            for (int j = 0; j < FN; ++j) acc[p][i][j] = mfma16x16x4(av[i], bv[j], acc[p][i][j]);
                    }
                }
            }
            if (more) store(cur ^ 1);
            if (!INV && s + 2 < nstages) {
#pragma unroll
                for (int v = 0; v < NM; ++v) {
                    mp1[v] = mp2[v];
                    mq1[v] = mq2[v];
                }
            }
            __syncthreads();
        }
    };
    static_assert(FM == 1 || FM == 2, "one or two row fragments per wave");
    // the inverse's ragged rows are few (2 % of its MFMAs against 6 % in the
    // direct): whole waves only, which keeps its registers within the two
    // blocks per CU
    if (nfa == FM || (INV && nfa > 0))
        kloop(std::integral_constant<int, FM>{});
    else if (!INV && nfa == 1)
        kloop(std::integral_constant<int, 1>{});
    else
        kloop(std::integral_constant<int, 0>{});

    if constexpr (INV) {
        T *four = (T *)a.out;
        // all rows' ring offsets first, so that their loads overlap
        RingPair ro[FM][4];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                int r = row0 + wr + i * 16 + acc_row<T>(lane, v);
                ro[i][v] = RingPair{-1, -1};
                if (r < b.R) ro[i][v] = a.ring_pair[b.j0 + r];
            }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const RingPair o = ro[i][v];
                if (o.n < 0) continue;
                T *fn = four + 2 * ((int64_t)o.n + m) * a.nfld;
                T *fs = four + 2 * ((int64_t)o.s + m) * a.nfld;
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    int c = col0 + wc + j * 16 + (lane & 15);
                    if (c < ncol) {
                        T s0 = acc[0][i][j][v], s1 = acc[1][i][j][v];
                        fn[c] = s0 + s1;
                        fs[c] = s0 - s1;
                    }
                }
            }
    } else {
        // direct scattered stores (staging through LDS measured slower for these
        // small tiles)
        T *spec = (T *)a.out;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        int k = row0 + wr + i * 16 + acc_row<T>(lane, v);
                        int c = col0 + wc + j * 16 + (lane & 15);
                        int nrel = p + 2 * k;
                        if (m + nrel <= a.trunc && c < ncol) {
                            T val = acc[p][i][j][v];
                            if (m == 0 && (c & 1)) val = 0;
                            spec[2 * ((int64_t)(c >> 1) * a.nspec + sb + nrel) + (c & 1)] = val;
                        }
                    }
    }
}

// ---------------------------------------------------------------------------
// Few fields, FP64 / FP32: at most 16 FN real columns.  With so few columns the
// table is most of the bytes and each entry is used once, so it goes from
// memory straight to the MFMA operand registers: lane l of a wave reads
// 16 bytes (VEC consecutive rows) of table row kappa = 4 s + l / 16, and
// component v of the load is the A operand of the MFMA over rows VEC (l % 16)
// + v.  A block covers 64 rows and both parities; its four waves take every
// fourth K step (a small plan has few tiles, so the K range is split over the
// block, and no barrier stands in the K loop) and their sums meet in LDS in a
// fixed order.  Bound by the table's bytes: T1279 on O1280, 3 fields, FP32
// inverse 1.33 -> 0.78 ms, direct 1.43 -> 0.75 ms (3.3 GB of table entries,
// 4.2-4.4 TB/s) against 128 x 128 tiles, where 122 of 128 columns were
// padding; T255, 7 fields 30 -> 14 and 47 -> 16 us; T639, 8 fields, FP64 240 ->
// 227 and 276 -> 235 us (0.9 GB).
// ---------------------------------------------------------------------------
constexpr int kNarrowWaves = 4;
// two complex values at the alignment of one
template <typename T>
struct __attribute__((aligned(2 * sizeof(T)))) Vec4 {
    T a, b, c, d;
};

template <typename T, int FN, bool INV>
__global__ __launch_bounds__(64 * kNarrowWaves) void k_leg_narrow(GemmArgs a)
{
    constexpr int VEC = 16 / sizeof(T), NL = 4 / VEC;  // rows per load, loads per K step and parity
    constexpr int NW = kNarrowWaves, BM = kNarrowRows, U = sizeof(T) == 4 ? 4 : 2;
    // INV: columns of one pair of fragments, real parts of NF fields then (in
    // the upper half of the lanes, or in the second fragment) their imaginary
    // parts, so that a lane's one load serves both parities (and both parts)
    constexpr int NF = FN == 1 ? 8 : 16, NP = FN == 1 ? 1 : FN / 2, LDC = INV ? 2 * NF + 2 : 18;
    typedef typename Acc<T>::type V;
    typedef T VecT __attribute__((ext_vector_type(VEC)));
    __shared__ __attribute__((aligned(16))) T red[NW][INV ? 1 : 2][BM][LDC];

    const GemmItem it = a.items[xcd_remap(blockIdx.x, gridDim.x)];
    if (it.m < 0) return;
    const int m = it.m;
    const MBlock b = a.mb[m];
    const int row0 = it.tr * BM, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4, ncol = 2 * a.nfld;
    const int64_t pstride = (int64_t)b.Kp * b.Rp;
    const int lda_g = INV ? b.Rp : b.Kp;
    const T *A0 = (const T *)a.tab + b.off + (int64_t)lk * lda_g + row0 + VEC * lr;
    const int64_t sb = spec_base(a.trunc, m);
    const int kend = INV ? b.K0 : b.R, nsteps = (kend + 3) / 4;

    V acc[2][4][FN];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[p][v][j] = V{};

    for (int s0 = wave; s0 < nsteps; s0 += NW * U) {
        VecT av[U][2][NL];
        T bv[U][2][FN];
        RingPair ro[U];
        T rq[U];
        if constexpr (!INV) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = 4 * (s0 + u * NW) + lk;
                ro[u] = RingPair{-1, -1};
                rq[u] = T(0);
                if (r < b.R) {
                    ro[u] = a.ring_pair[b.j0 + r];
                    rq[u] = a.adjoint ? T(1) : ((const T *)a.ring_q)[b.j0 + r];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u * NW;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    av[u][p][l] = VecT{};
                    if (s < nsteps)  // wave-uniform; the tables are padded past kend
                        av[u][p][l] = *reinterpret_cast<const VecT *>(A0 + p * pstride + (int64_t)(4 * s) * lda_g +
                                                                      16 * VEC * l);
                }
            if constexpr (INV) {
                const int nrel = 2 * (4 * s + lk);
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const int f = NF * j + (lr & (NF - 1));
                    const Vec2<T> *src = (const Vec2<T> *)a.in + (int64_t)f * a.nspec + sb + nrel;
                    Vec2<T> z0 = {T(0), T(0)}, z1 = {T(0), T(0)};
                    if (f < a.nfld && m + nrel + 1 <= a.trunc) {
                        const Vec4<T> z = *reinterpret_cast<const Vec4<T> *>(src);
                        z0 = Vec2<T>{z.a, z.b};
                        z1 = Vec2<T>{z.c, z.d};
                    } else if (f < a.nfld && m + nrel <= a.trunc) {
                        z0 = src[0];
                    }
                    // Im a^0_n is ignored
                    if (m == 0) z0.y = z1.y = T(0);
                    if constexpr (FN == 1) {
                        bv[u][0][0] = lr < NF ? z0.x : z0.y;
                        bv[u][1][0] = lr < NF ? z1.x : z1.y;
                    } else {
                        bv[u][0][2 * j] = z0.x;
                        bv[u][0][2 * j + 1] = z0.y;
                        bv[u][1][2 * j] = z1.x;
                        bv[u][1][2 * j + 1] = z1.y;
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const int c = 16 * j + lr;
                    bv[u][0][j] = T(0);
                    bv[u][1][j] = T(0);
                    if (ro[u].n >= 0 && c < ncol) {
                        const T *four = (const T *)a.in;
                        bv[u][0][j] = four[2 * ((int64_t)ro[u].n + m) * a.nfld + c];
                        bv[u][1][j] = four[2 * ((int64_t)ro[u].s + m) * a.nfld + c];
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                T b0 = bv[u][0][j], b1 = bv[u][1][j];
                if constexpr (!INV) {
                    // hemispheric fold
                    const T gn = b0, gs = b1;
                    b0 = rq[u] * (gn + gs);
                    b1 = rq[u] * (gn - gs);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    acc[0][v][j] = mfma16x16x4(av[u][0][v / VEC][v % VEC], b0, acc[0][v][j]);
                    acc[1][v][j] = mfma16x16x4(av[u][1][v / VEC][v % VEC], b1, acc[1][v][j]);
                }
            }
    }

    auto row = [&](int v, int t) { return 16 * VEC * (v / VEC) + VEC * acc_row<T>(lane, t) + v % VEC; };
    auto sum = [&](int p, int r, int c) {
        T x = red[0][p][r][c];
#pragma unroll
        for (int w = 1; w < NW; ++w) x += red[w][p][r][c];
        return x;
    };
    if constexpr (INV) {
        // the waves' sums, one pair of fragments and one hemisphere at a time:
        // runs over fields of each ring row
#pragma unroll
        for (int q = 0; q < 2 * NP; ++q) {
            const int hs = q & 1, j = q >> 1;
            if (NF * j >= a.nfld) break;
            if (q) __syncthreads();
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if constexpr (FN == 1) {
                        const T s0 = acc[0][v][0][t], s1 = acc[1][v][0][t];
                        red[wave][0][row(v, t)][2 * (lr & 7) + (lr >> 3)] = hs ? s0 - s1 : s0 + s1;
                    } else {
                        const T x0 = acc[0][v][2 * j][t], x1 = acc[1][v][2 * j][t];
                        const T y0 = acc[0][v][2 * j + 1][t], y1 = acc[1][v][2 * j + 1][t];
                        *reinterpret_cast<Vec2<T> *>(&red[wave][0][row(v, t)][2 * lr]) =
                            hs ? Vec2<T>{x0 - x1, y0 - y1} : Vec2<T>{x0 + x1, y0 + y1};
                    }
                }
            __syncthreads();
#pragma unroll
            for (int i = tid; i < BM * NF; i += 64 * NW) {
                const int r = i / NF, fl = i % NF, f = NF * j + fl;
                if (row0 + r >= b.R || f >= a.nfld) continue;
                const RingPair o = a.ring_pair[b.j0 + row0 + r];
                ((Vec2<T> *)a.out)[((int64_t)(hs ? o.s : o.n) + m) * a.nfld + f] =
                    Vec2<T>{sum(0, r, 2 * fl), sum(0, r, 2 * fl + 1)};
            }
        }
    } else {
        // the waves' sums, 16 columns at a time: runs of n of one field
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            if (16 * j >= ncol) break;
            if (j) __syncthreads();
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int t = 0; t < 4; ++t) red[wave][p][row(v, t)][lr] = acc[p][v][j][t];
            __syncthreads();
#pragma unroll
            for (int i = tid; i < 2 * BM * 8; i += 64 * NW) {
                const int fl = i / (2 * BM), nr = i % (2 * BM), f = 8 * j + fl, nrel = 2 * row0 + nr;
                if (f >= a.nfld || m + nrel > a.trunc) continue;
                const T x = sum(nr & 1, nr >> 1, 2 * fl);
                const T y = m == 0 ? T(0) : sum(nr & 1, nr >> 1, 2 * fl + 1);
                ((Vec2<T> *)a.out)[(int64_t)f * a.nspec + sb + nrel] = Vec2<T>{x, y};
            }
        }
    }
}

// ---------------------------------------------------------------------------
// FP32 and the split forms, on the half-precision matrix cores with FP32
// accumulation.  Each operand is a sum of 16-bit pieces and a tile product is
// the MFMAs of the piece pairs that matter, smallest first:
//   SHTX_FP32    three bfloat16 pieces, 8 + 8 + 8 significand bits: a float
//                exactly, if it is not below 2^-110, where pieces fall under
//                bfloat16's smallest value; the six products down to 2^-16
//                of the largest (those left out come to 2^-24.0 of it at
//                most, 2^-27 on average; FP32 rounds each sum to 2^-24)
//   SHTX_BF16X3  bfloat16 hi + lo, three products (lo lo is dropped)
//   SHTX_FP16X3  IEEE half hi + lo, three products
// The split forms' table is stored in pieces, scaled by 2^e_m per m; FP32's as
// floats, scaled by 2^16 (its smallest entries have whole pieces), which are cut
// here like the data operand, once per block and stage.  IEEE half has a 5-bit
// exponent, so its data operand is also scaled per field by 2^E_f, chosen from
// a bound on the field's largest value; bfloat16 has the FP32 exponent range
// and needs no data scale.  A tile of the FP32 form that meets a smaller value than its
// pieces hold, one that is not finite, or a sum beyond 2^112 runs again on the
// single-precision matrix cores: only there do such values keep 24 bits.  In
// the split forms an infinite value gives NaN.
//
// 32x32x16 MFMA: lane l supplies A[l%32][8(l/32)..+7] and B[8(l/32)..+7][l%32]
// and holds D[8(v/4) + 4(l/32) + v%4][l%32], v = 0..15.  Both operands come in
// units of 16 bytes, 8 consecutive kappa of one row: the table is laid out in
// memory as planes [piece][parity][kappa / 8][row] of units (FP32: of 32-byte
// units without pieces), so a stage's loads and LDS writes are runs of units
// (no transposition, no bank conflicts), and LDS holds one 16-deep stage in
// the same order.
//
// A block covers 64 FI rows and 32 FJ fields (64 FJ columns), both parities, in
// four waves of 32 fields (real and imaginary parts: two column fragments) and
// the 32-row fragments wr, wr + WR, ... of the tile; the next stage's loads are
// in flight over the MFMAs.
//
// O1280, 411 fields, against the kernels before (16x16x4 FP32 MFMA; split
// operands re-staged by field): FP32 inverse 13.4 -> 9.95 ms, direct 13.6 -> 11.3;
// BF16x3 8.3 -> 6.9 and 8.8 -> 7.6; T399, 137 fields, FP32 244 -> 176 and 285 ->
// 224 us; T2799 on 4200 x 8400 points, 120 fields, 35.8 -> 25.0 and 37.5 -> 28.7 ms.
// (With the data cut instead of rounded to its first piece, no look for values
// that pieces do not hold and the FP32 table in pieces: 9.7 and 11.0.)  Of the
// FP32 inverse's 9.8 ms then, found by leaving out one part at a
// time: MFMAs 2.7, operand loads 2.7, conversion and LDS stores 1.4, output and
// block start 2.3 (8.1 GB written); the parts add up instead of overlapping
// although two blocks share a CU, at a clock that falls to 2.0 GHz.
// ---------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
// vector loads and stores at 8-byte aligned addresses (vector memory
// instructions need only 4-byte alignment)
typedef float f32x4a8 __attribute__((ext_vector_type(4), aligned(8)));

// From this magnitude on a float is the sum of three bfloat16 pieces: its last
// bit is bfloat16's smallest value, 2^-133, or more.
constexpr float kPiecesHold = 0x1p-110f;

// Two floats -> packed pieces, most significant first.  Residuals must be taken
// against the very bits that are stored.  Left to itself the compiler
// re-derives hi for that subtraction from the product that produced x, by
// another instruction (a mixed-precision FMA rounding the exact product to
// half once) whose result differs from the stored hi wherever the two
// roundings disagree; hi + lo is then off by a unit of hi.  An empty asm
// statement makes the stored bits opaque, so the residual is computed from
// them.  All pieces are rounded to nearest: with the FP32 form's leading one cut
// instead, the products left out reached twice as much (2^-23 of a product).
// A value near the largest float rounds to an infinite piece, and its sums to
// NaN: the tile runs again.  `least` takes the smallest magnitude
// seen (FP32 form).
template <int FORM>
__device__ inline void split_pair(float x0, float x1, unsigned *w, float &least)
{
    if constexpr (FORM == SHTX_FP16X3) {
        unsigned hb = __builtin_bit_cast(unsigned, f16x2{(_Float16)x0, (_Float16)x1});
        asm("" : "+v"(hb));
        const f16x2 h = __builtin_bit_cast(f16x2, hb);
        w[0] = hb;
        w[1] = __builtin_bit_cast(unsigned, f16x2{(_Float16)(x0 - (float)h[0]), (_Float16)(x1 - (float)h[1])});
    } else {
        float r0 = x0, r1 = x1;
        // a piece of both, which leaves the rest in r0 and r1
        auto piece = [&]() __attribute__((always_inline)) {
            unsigned hb = __builtin_bit_cast(unsigned, bf16x2{(__bf16)r0, (__bf16)r1});
            asm("" : "+v"(hb));
            r0 -= __uint_as_float(hb << 16);
            r1 -= __uint_as_float(hb & 0xffff0000u);
            return hb;
        };
        w[0] = piece();
        if constexpr (FORM == SHTX_FP32) {
            // one instruction (fminf would first quiet its operands)
            asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(least) : "v"(x0), "v"(x1));
            w[1] = piece();
        }
        w[split_pieces(FORM) - 1] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)r0, (__bf16)r1});
    }
}

// 32x32x2 MFMA on floats: lane l supplies A[l%32][l/32] and B[l/32][l%32]; the
// result is laid out as that of the 16-bit forms.
__device__ inline f32x16 mfma32x32x2(float a, float b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Half t (0: low) of a word as the high half of a float's bits.
__device__ inline float piece_float(unsigned w, int t) { return __uint_as_float(t ? w & 0xffff0000u : w << 16); }

template <int FORM>
__device__ inline f32x16 mfma_split(u32x4 a, u32x4 b, f32x16 c)
{
    if constexpr (FORM == SHTX_FP16X3)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c,
                                                      0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                       c, 0, 0, 0);
}

// Exponent E_f of field f's data operand in the half form: with the field's
// largest magnitude times `bound` (a bound on the operand's entries) equal to
// x 2^X, x in [1/2, 1), E_f = 14 - X puts the bound in [2^13, 2^14); 0 for an
// all-zero field.
__device__ inline int field_exp(const unsigned *fmax, int f, float bound)
{
    const float mx = __uint_as_float(fmax[f]) * bound;
    if (!(mx > 0.f)) return 0;
    int X;
    (void)frexpf(mx, &X);
    return 14 - X;
}

// Transposes a quad of lanes' 4 x 4 values in registers: lane q's x[t] becomes
// lane t's x[q] (odd, upper: bits 0 and 1 of the lane index).
__device__ inline void quad_transpose(float *x, bool odd, bool upper)
{
    auto swap = [](float mine, auto ctrl) {
        return __uint_as_float(
            __builtin_amdgcn_mov_dpp(__float_as_uint(mine), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    // quad_perm [1, 0, 3, 2] and [2, 3, 0, 1]
    typedef std::integral_constant<int, 0xB1> xor1;
    typedef std::integral_constant<int, 0x4E> xor2;
#pragma unroll
    for (int t = 0; t < 4; t += 2) {
        const float r = swap(odd ? x[t] : x[t + 1], xor1{});
        x[t] = odd ? r : x[t];
        x[t + 1] = odd ? x[t + 1] : r;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const float r = swap(upper ? x[t] : x[t + 2], xor2{});
        x[t] = upper ? r : x[t];
        x[t + 2] = upper ? x[t + 2] : r;
    }
}

template <int FORM, int FI, int FJ, bool INV>
__global__ __launch_bounds__(256, FI * FJ == 4 ? 2 : 3) void k_leg_split(GemmArgs a)
{
    constexpr bool CUT = FORM == SHTX_FP32;  // table units of floats, cut on their way to LDS
    constexpr bool F16 = FORM == SHTX_FP16X3;
    constexpr int NP = split_pieces(FORM), BM = 64 * FI, BN = 64 * FJ, NF = 32 * FJ, BK = 16;
    constexpr int WR = 4 / FJ, NI = BM / (32 * WR);  // waves over the rows, row fragments per wave
    // units of an LDS plane: the rows of A; of B the real parts at 0 and the
    // imaginary ones at URI.  The offsets between parts and parities put the
    // four units that a quad of lanes stores on different banks.
    constexpr int UA = BM, URI = NF + 8, UB = URI + NF + 2, PA = NP * 4 * UA, PB = NP * 4 * UB;
    // the direct form stages its output in the same LDS: 2 BM + 1 complex
    // values of 32 fields
    constexpr int NSTAGE = INV ? 0 : 32 * (2 * BM + 1) / 2;
    constexpr int NSMEM = PA + PB > NSTAGE ? PA + PB : NSTAGE;
    constexpr int NTP = CUT ? 2 : NP;  // 16-byte loads of a table unit: halves or pieces
    constexpr int NA = NTP * FI;       // and of a stage's units, per thread
    __shared__ u32x4 smem[NSMEM];
    __shared__ int wave_lost[4];
    u32x4 *As = smem, *Bs = smem + PA;

    const GemmItem it = a.items[xcd_remap(blockIdx.x, gridDim.x)];
    if (it.m < 0) return;
    const int m = it.m;
    const MBlock b = a.mb[m];
    const int row0 = it.tr * BM, f0 = it.tc * NF;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / FJ, fj = wave % FJ;
    const int64_t sb = spec_base(a.trunc, m);
    const int kend = INV ? b.K0 : b.R, nstages = (kend + BK - 1) / BK;
    // the m block's table through a buffer descriptor: a unit's plane and row
    // are a scalar offset, the only vector address is the lane
    const int rows = INV ? b.Rp : b.Kp, chunks = (INV ? b.Kp : b.Rp) / 8;
    const int64_t tab_units = (int64_t)NTP * 2 * chunks * rows;
    const auto tab = __builtin_amdgcn_make_buffer_rsrc((void *)((const u32x4 *)a.tab + b.off / 8 * NTP), 0,
                                                       (int)(tab_units * 16), 0x00027000);
    // This thread's share of B.  INV: a quad of lanes takes the 16 kappa of one
    // field, reading 64 contiguous bytes at a time, and transposes them so that
    // lane q holds one parity and part (q / 2, q % 2) of every kappa.  DIR:
    // rings 8 kh .. + 7 of column t, both hemispheres.
    const bool bon = FJ == 2 || wave < 2;
    const int bf = INV ? tid >> 2 : (tid & (BN - 1)) >> 1, kh = FJ == 2 ? wave >> 1 : wave & 1;
    const int bp = tid >> 1 & 1, bri = tid & 1;
    const int bfc = min(f0 + bf, a.nfld - 1);  // past the last field: repeated, not stored
    float scale = 1.f;
    if constexpr (F16) scale = ldexpf(1.f, field_exp(a.fmax, bfc, a.dbound));
    // INV: the ring offsets of one row per thread, for the epilogue
    RingPair orow = {0, 0};
    if (INV && tid < BM && row0 + tid < b.R) orow = a.ring_pair[b.j0 + row0 + tid];

    u32x4 ra[NA];
    f32x4 rb[4];
    float rn[8], rs[8];
    // DIR: lane q < 8 holds ring 8 kh + q of the next load, fetched a stage ahead
    RingPair mp = {0, 0};
    float mq = 0.f, q1[8];
    auto meta = [&](int kk) __attribute__((always_inline)) {
        // past the last ring: repeated (the table's padding is zero); nothing here
        // may wait for these loads, which would wait for the operands' too
        const int j = b.j0 + min(kk + 8 * kh + (lane & 7), b.R - 1);
        mp = a.ring_pair[j];
        mq = ((const float *)a.ring_q)[j];
    };
    auto load = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            // wave-loads of 64 rows: (plane, row half)
            const int q = wave + 4 * (CUT ? i / 2 : i), half = q % FI, kc = q / FI & 1, pp = q / (2 * FI);
            const int unit = (pp * chunks + kk / 8 + kc) * rows + row0 + 64 * half;
            ra[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  tab, CUT ? 32 * lane : 16 * lane,
                                                  CUT ? 32 * unit + 16 * (i & 1) : 16 * unit, 0));
        }
        if (!bon) return;
        if constexpr (INV) {
            const float2 *src = (const float2 *)a.in + (int64_t)bfc * a.nspec + sb;
            const int nrel = 2 * (kk + (tid & 3));
            if (m + 2 * kk + 2 * BK - 1 <= a.trunc) {
#pragma unroll
                for (int i = 0; i < 4; ++i) rb[i] = *reinterpret_cast<const f32x4a8 *>(src + nrel + 8 * i);
            } else {
                // past the last degree: repeated (the table's padding is zero)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float2 z0 = src[min(nrel + 8 * i, a.trunc - m)], z1 = src[min(nrel + 8 * i + 1, a.trunc - m)];
                    rb[i] = f32x4{z0.x, z0.y, z1.x, z1.y};
                }
            }
        } else {
            const float *four = (const float *)a.in;
            const unsigned c = 2 * bfc + (tid & 1);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int on = __builtin_amdgcn_readlane(mp.n, q), os = __builtin_amdgcn_readlane(mp.s, q);
                rn[q] = (four + 2 * ((int64_t)on + m) * a.nfld)[c];
                rs[q] = (four + 2 * ((int64_t)os + m) * a.nfld)[c];
                const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(mq), q));
                q1[q] = a.adjoint ? 1.f : w;
            }
        }
    };
    uint64_t lost = 0;  // lanes that met a value which its pieces do not hold
    auto note = [&](float x) __attribute__((always_inline)) {
        lost |= __builtin_amdgcn_ballot_w64(x != 0.f && fabsf(x) < kPiecesHold);
    };
    // WHOLE: the data operand's floats uncut, high halves in the plane of the
    // first piece and low halves in that of the second
    auto store = [&](auto whole_c) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole_c)::value;
        constexpr int NB = WHOLE ? 2 : NP;
        float least = 1.f;
        auto cut = [&](float x0, float x1, unsigned *w) __attribute__((always_inline)) {
            if constexpr (WHOLE) {
                w[0] = __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);
                w[1] = __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x05040100u);
            } else {
                split_pair<FORM>(x0, x1, w, least);
            }
        };
        if constexpr (CUT) {
#pragma unroll
            for (int i = 0; i < FI; ++i) {
                unsigned w[4][NP];
                float any = 1.f;  // the scale leaves no entry that pieces would not hold
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    split_pair<FORM>(__uint_as_float(ra[2 * i + t / 2][2 * (t & 1)]),
                                     __uint_as_float(ra[2 * i + t / 2][2 * (t & 1) + 1]), w[t], any);
#pragma unroll
                for (int h = 0; h < NP; ++h)
                    As[h * 4 * UA + (wave + 4 * i) * 64 + lane] = u32x4{w[0][h], w[1][h], w[2][h], w[3][h]};
            }
        } else {
#pragma unroll
            for (int i = 0; i < NA; ++i) As[(wave + 4 * i) * 64 + lane] = ra[i];
        }
        if (!bon) return;
        if constexpr (INV) {
            // kappa 4 i + q of lane q -> kappa 4 i .. + 3 of lane q's value
            unsigned w[8][NP];
            const bool off = bri && m == 0;  // Im a^0_n is ignored
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float x[4] = {rb[i][0], rb[i][1], rb[i][2], rb[i][3]};
                quad_transpose(x, bri, bp);
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    cut(off ? 0.f : x[2 * t] * scale, off ? 0.f : x[2 * t + 1] * scale, w[2 * i + t]);
            }
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) {
                u32x4 *dst = Bs + (2 * bp + kc) * UB + bri * URI + bf;
#pragma unroll
                for (int h = 0; h < NB; ++h)
                    dst[h * 4 * UB] = u32x4{w[4 * kc][h], w[4 * kc + 1][h], w[4 * kc + 2][h], w[4 * kc + 3][h]};
            }
            if (FORM == SHTX_FP32 && !WHOLE && __builtin_expect(__builtin_amdgcn_ballot_w64(least < kPiecesHold) != 0, 0)) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int t = 0; t < 4; ++t) note(m == 0 && (t & 1) ? 0.f : rb[i][t]);
            }
        } else {
            // hemispheric fold: parity 0 takes q (north + south), parity 1 q (north - south)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                unsigned w[4][NP];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float x[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int q = 2 * i + t;
                        x[t] = (q1[q] * scale) * (p ? rn[q] - rs[q] : rn[q] + rs[q]);
                    }
                    cut(x[0], x[1], w[i]);
                }
                u32x4 *dst = Bs + (2 * p + kh) * UB + (tid & 1) * URI + bf;
#pragma unroll
                for (int h = 0; h < NB; ++h) dst[h * 4 * UB] = u32x4{w[0][h], w[1][h], w[2][h], w[3][h]};
            }
            if (FORM == SHTX_FP32 && !WHOLE && __builtin_expect(__builtin_amdgcn_ballot_w64(least < kPiecesHold) != 0, 0)) {
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    note(q1[q] * (rn[q] + rs[q]));
                    note(q1[q] * (rn[q] - rs[q]));
                }
            }
        }
    };

    f32x16 acc[2][NI][2];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[p][i][j][v] = 0.f;
    };
    clear();

    auto kloop = [&](auto ni_c) __attribute__((always_inline)) {
        constexpr int NA_I = decltype(ni_c)::value;  // row fragments in use
        if (nstages == 0) return;                    // a wavenumber that no ring carries
        if (!INV) meta(0);
        load(0);
        if (!INV) meta(BK);
        for (int s = 0; s < nstages; ++s) {
            store(std::false_type{});
            __syncthreads();
            if (s + 1 < nstages) load((s + 1) * BK);  // in flight during the MFMAs
            if (!INV) meta((s + 2) * BK);
            if constexpr (NA_I > 0) {
                const int kc = lane >> 5, ln = lane & 31;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    u32x4 av[NA_I][NP], bv[2][NP];
#pragma unroll
                    for (int h = 0; h < NP; ++h) {
#pragma unroll
                        for (int i = 0; i < NA_I; ++i)
                            av[i][h] = As[((2 * h + p) * 2 + kc) * UA + 32 * (WR * i + wr) + ln];
#pragma unroll
                        for (int j = 0; j < 2; ++j) bv[j][h] = Bs[((2 * h + p) * 2 + kc) * UB + j * URI + 32 * fj + ln];
                    }
                    // piece pairs (x, y) with x + y < NP, smallest products first
#pragma unroll
                    for (int t = NP - 1; t >= 0; --t)
#pragma unroll
                        for (int x = t; x >= 0; --x)
#pragma unroll
                            for (int i = 0; i < NA_I; ++i)
#pragma unroll
                                for (int j = 0; j < 2; ++j)
                                    acc[p][i][j] = mfma_split<FORM>(av[i][x], bv[j][t - x], acc[p][i][j]);
                }
            }
            __syncthreads();
        }
    };
    // Row fragments of this wave that hold data (wave-uniform; none when its
    // fields are past the last): the others skip their LDS reads and MFMAs,
    // while the wave still loads and stores its share.  One copy of the K loop
    // per count keeps the accumulators in place.
    const int f = f0 + 32 * fj + (lane & 31);
    const int nrow = f0 + 32 * fj < a.nfld ? (INV ? b.R : b.K0) - row0 - 32 * wr : 0;
    if (nrow <= 0)
        kloop(std::integral_constant<int, 0>{});
    else if (NI == 1 || nrow > 32 * WR)
        kloop(std::integral_constant<int, NI>{});
    else
        kloop(std::integral_constant<int, 1>{});

    // INV: the two parities' sums become the two hemispheres' (FP32: without the
    // table's scale, so that they are finite wherever those are)
    auto fold = [&](float unit) __attribute__((always_inline)) {
        if constexpr (!INV) return;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float x0 = FORM == SHTX_FP32 ? unit * acc[0][i][j][v] : acc[0][i][j][v];
                    const float x1 = acc[1][i][j][v];
                    acc[0][i][j][v] = FORM == SHTX_FP32 ? fmaf(x1, unit, x0) : x0 + x1;
                    acc[1][i][j][v] = FORM == SHTX_FP32 ? fmaf(x1, -unit, x0) : x0 - x1;
                }
    };
    // A tile that met a value which is not the sum of its pieces (below 2^-110, or
    // not finite), or whose sums left the range that the table's scale leaves,
    // runs once more, as plain single-precision products on the FP32 matrix
    // cores (the table's entries are the sums of their pieces; 1/5 of the rate,
    // but no ordinary field comes here).  All four waves go or none.
    float unit = FORM == SHTX_FP32 ? 1.f / kF32TableScale : 1.f;
    fold(unit);
    if constexpr (FORM == SHTX_FP32) {
        // the sum of all is finite only if each is (an inverse tile's northern
        // sums alone: they are finite only if both parities' are)
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < (INV ? 1 : 2); ++p)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) sum[v & 3] += acc[p][i][j][v];
        lost |= __builtin_amdgcn_ballot_w64(!__builtin_isfinite((sum[0] + sum[1]) + (sum[2] + sum[3])));
        if (lane == 0) wave_lost[wave] = lost != 0;
        __syncthreads();
        if (__builtin_expect(wave_lost[0] | wave_lost[1] | wave_lost[2] | wave_lost[3], 0)) {
            unit = 1.f;
            clear();
            for (int s = 0; s < nstages; ++s) {
                if (!INV) meta(s * BK);
                load(s * BK);
                store(std::true_type{});
                __syncthreads();
                const int kc = lane >> 5, ln = lane & 31;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    u32x4 av[NI][NP], bv[2][2];
#pragma unroll
                    for (int h = 0; h < NP; ++h)
#pragma unroll
                        for (int i = 0; i < NI; ++i)
                            av[i][h] = As[((2 * h + p) * 2 + kc) * UA + 32 * (WR * i + wr) + ln];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int j = 0; j < 2; ++j) bv[j][h] = Bs[((2 * h + p) * 2 + kc) * UB + j * URI + 32 * fj + ln];
                    // kappa t of the lower half of the lanes with kappa 8 + t of the upper
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        float x[NI], y[2];
#pragma unroll
                        for (int i = 0; i < NI; ++i) {
                            float z = piece_float(av[i][NP - 1][t / 2], t & 1);
#pragma unroll
                            for (int h = NP - 2; h >= 0; --h) z += piece_float(av[i][h][t / 2], t & 1);
                            x[i] = z * (1.f / kF32TableScale);
                        }
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            y[j] = __uint_as_float(__builtin_amdgcn_perm(bv[j][0][t / 2], bv[j][1][t / 2],
                                                                         t & 1 ? 0x07060302u : 0x05040100u));
#pragma unroll
                        for (int i = 0; i < NI; ++i)
#pragma unroll
                            for (int j = 0; j < 2; ++j) acc[p][i][j] = mfma32x32x2(x[i], y[j], acc[p][i][j]);
                    }
                }
                __syncthreads();
            }
            fold(unit);
        }
    }

    auto frag_row = [&](int i, int v) { return 32 * (WR * i + wr) + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); };
    // undoes the scales of the table block and of this lane's field
    int e = 0;
    if constexpr (FORM != SHTX_FP32) e = -(b.e + (F16 ? field_exp(a.fmax, min(f, a.nfld - 1), a.dbound) : 0));
    auto unscale = [&](float x) { return FORM != SHTX_FP32 ? ldexpf(x, e) : INV ? x : x * unit; };
    if constexpr (INV) {
        // a lane holds its field's real and imaginary part of each row: runs of
        // 32 fields straight to both hemispheres' rows
        RingPair *orows = reinterpret_cast<RingPair *>(smem);
        if (tid < BM) orows[tid] = orow;
        __syncthreads();
        float2 *four = (float2 *)a.out;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = frag_row(i, v);
                const RingPair o = orows[r];
                if (row0 + r >= b.R || f >= a.nfld) continue;
                four[((int64_t)o.n + m) * a.nfld + f] = float2{unscale(acc[0][i][0][v]), unscale(acc[0][i][1][v])};
                four[((int64_t)o.s + m) * a.nfld + f] = float2{unscale(acc[1][i][0][v]), unscale(acc[1][i][1][v])};
            }
    } else {
        // 32 fields at a time as [field][n], written as runs of n
        constexpr int RS = 2 * BM + 1;
        float2 *st = reinterpret_cast<float2 *>(smem);
        float2 *spec = (float2 *)a.out;
        const int nrel0 = 2 * row0, nvalid = min(2 * BM, a.trunc - m - nrel0 + 1);
#pragma unroll
        for (int h = 0; h < FJ; ++h) {
            if (h) __syncthreads();
            if (fj == h) {
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int i = 0; i < NI; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            st[(lane & 31) * RS + p + 2 * frag_row(i, v)] =
                                float2{unscale(acc[p][i][0][v]), m == 0 ? 0.f : unscale(acc[p][i][1][v])};
            }
            __syncthreads();
            for (int fl = wave; fl < 32; fl += 4) {
                if (f0 + h * 32 + fl >= a.nfld) break;
                float2 *dst = spec + (int64_t)(f0 + h * 32 + fl) * a.nspec + sb + nrel0;
                for (int nr = lane; nr < nvalid; nr += 64) dst[nr] = st[fl * RS + nr];
            }
        }
    }
}

GemmArgs make_args(const Plan &p, bool inverse_shape, const void *in, void *out, bool adjoint, unsigned *fmax)
{
    GemmArgs a{};
    a.mb = p.d_mb;
    a.items = inverse_shape ? p.d_inv_items : p.d_dir_items;
    a.ring_pair = p.d_ring_pair;
    a.ring_q = p.d_ring_q;
    a.in = in;
    a.out = out;
    a.trunc = p.trunc;
    a.nlat = p.nlat;
    a.nfld = p.nfld;
    a.adjoint = adjoint ? 1 : 0;
    a.nspec = p.nspec;
    a.tab = inverse_shape ? p.d_tab_inv : p.d_tab_dir;
    // the inverse-shaped launch splits spectral coefficients (bounded by the
    // field maximum itself); the direct-shaped one splits q_r (G_north +-
    // G_south), bounded by 2 max_r q_r times the largest Fourier value
    a.fmax = fmax;
    a.dbound = inverse_shape ? 1.f : (float)(2.0 * (adjoint ? 1.0 : p.qmax));
    return a;
}

// Host check that every tile of a work list reads and writes inside the table, Fourier and spectral arrays for the
// given tile sizes.  Run when a plan's work lists are built, not per launch.
bool check_items(const Plan &p, const std::vector<GemmItem> &items, bool inverse_shape, int bm, int bn, int bk)
{
    if (items.empty() || items.size() % kXcds) return false;
    int ncol = 2 * p.nfld;
    for (const GemmItem &it : items) {
        if (it.m < 0) continue;
        if (it.m > p.trunc) return false;
        const MBlock &b = p.mb[it.m];
        if (it.tc < 0 || it.tc * bn >= ncol) return false;
        if (inverse_shape) {
            if (it.tr < 0 || it.tr * bm >= b.R || (it.tr + 1) * bm > b.Rp) return false;
            if ((int64_t)((b.K0 + bk - 1) / bk) * bk > b.Kp) return false;
        } else {
            if (it.tr < 0 || it.tr * bm >= b.K0 || (it.tr + 1) * bm > b.Kp) return false;
            if ((int64_t)((b.R + bk - 1) / bk) * bk > b.Rp) return false;
        }
        if (b.j0 + b.R > p.nlat / 2) return false;
    }
    return true;
}

bool check_work_list(const Plan &p, const std::vector<GemmItem> &items, bool inverse_shape, int bm, int bn, int bk)
{
    const bool ok = check_items(p, items, inverse_shape, bm, bn, bk);
    if (!ok && std::getenv("SHTX_DEBUG"))
        std::fprintf(stderr, "shtx: Legendre GEMM work-list check failed (%s)\n", inverse_shape ? "inverse" : "direct");
    return ok;
}

// The few-fields kernel with fn column fragments (gemm_narrow).
template <typename T, bool INV>
hipError_t launch_narrow(const GemmArgs &a, int fn, int grid, hipStream_t s)
{
    if (fn == 1) {
        k_leg_narrow<T, 1, INV><<<grid, 64 * kNarrowWaves, 0, s>>>(a);
        return hipGetLastError();
    }
    if constexpr (sizeof(T) == 4) {
        if (fn == 2) {
            k_leg_narrow<T, 2, INV><<<grid, 64 * kNarrowWaves, 0, s>>>(a);
            return hipGetLastError();
        }
        if constexpr (!INV) {
            if (fn == 4) {
                k_leg_narrow<T, 4, INV><<<grid, 64 * kNarrowWaves, 0, s>>>(a);
                return hipGetLastError();
            }
        }
    }
    return hipErrorInvalidValue;
}

template <bool INV>
hipError_t launch_fp64(const Plan &p, const GemmArgs &a, int bm, int bn, hipStream_t s)
{
    // the work lists were checked against these shapes when they were built
    const int grid = (int)(INV ? p.inv_items : p.dir_items).size(), narrow = INV ? p.inv_narrow : p.dir_narrow;
    if (!p.shapes_ok || grid < 1) return hipErrorInvalidValue;
    if (narrow) return launch_narrow<double, INV>(a, narrow, grid, s);
#define SHTX_TILE(BM, BN, NW)                                              \
    if (bm == BM && bn == BN) {                                            \
        k_leg_mfma<double, BM, BN, 16, INV, NW><<<grid, 64 * NW, 0, s>>>(a); \
        return hipGetLastError();                                          \
    }
    SHTX_TILE(64, 64, 8)
    SHTX_TILE(32, 64, 8)
    SHTX_TILE(64, 32, 4)
#undef SHTX_TILE
    return hipErrorInvalidValue;
}

// Largest magnitude of each field's spectral coefficients (Re and Im of
// every a_n^m except Im a_n^0, which the transforms ignore), as float bits:
// the bound from which the half form scales the inverse-shaped GEMM's data
// operand.  Blocks (chunk, field) each take a contiguous chunk of one
// field's coefficients and fold their maximum into fmax[f] with an atomic
// max (non-negative floats order as their bits), after k_clear_u32 has
// zeroed it; the maximum does not depend on the order.
constexpr int kAbsmaxChunks = 8;

__global__ void k_clear_u32(unsigned *x, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0u;
}

__global__ __launch_bounds__(1024) void k_spec_absmax(const float2 *spec, int64_t nspec, int trunc, unsigned *fmax)
{
    __shared__ float red[16];
    const int f = blockIdx.y;
    const int64_t chunk = (nspec + kAbsmaxChunks - 1) / kAbsmaxChunks;
    const int64_t i0 = blockIdx.x * chunk, i1 = min(nspec, i0 + chunk);
    const float2 *row = spec + (int64_t)f * nspec;
    float mx = 0.f;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 1024) {
        const float2 z = row[i];
        mx = fmaxf(mx, fabsf(z.x));
        if (i > trunc) mx = fmaxf(mx, fabsf(z.y));  // index i <= N is m = 0
    }
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int w = 0; w < 16; ++w) t = fmaxf(t, red[w]);
        atomicMax(fmax + f, __float_as_uint(t));
    }
}

template <int FORM, bool INV>
hipError_t launch_split(const Plan &p, const GemmArgs &a, int bm, int bn, hipStream_t s)
{
    const int grid = (int)(INV ? p.inv_items : p.dir_items).size();
    if (!p.shapes_ok || grid < 1) return hipErrorInvalidValue;
    if (bm == 128 && bn == 128) {
        k_leg_split<FORM, 2, 2, INV><<<grid, 256, 0, s>>>(a);
    } else if (bm == 64 && bn == 128) {
        k_leg_split<FORM, 1, 2, INV><<<grid, 256, 0, s>>>(a);
    } else if constexpr (FORM == SHTX_FP32) {
        if (bm != 128 || bn != 64) return hipErrorInvalidValue;
        k_leg_split<FORM, 2, 1, INV><<<grid, 256, 0, s>>>(a);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool INV>
hipError_t launch_fp32(const Plan &p, const GemmArgs &a, int bm, int bn, hipStream_t s)
{
    const int narrow = INV ? p.inv_narrow : p.dir_narrow;
    if (!narrow) return launch_split<SHTX_FP32, INV>(p, a, bm, bn, s);
    if (!p.shapes_ok) return hipErrorInvalidValue;
    return launch_narrow<float, INV>(a, narrow, (int)(INV ? p.inv_items : p.dir_items).size(), s);
}

}  // namespace

// Tile shapes with a kernel instantiation.
int gemm_tile_candidates(int prec, int *bm, int *bn, int max)
{
    static const int f32[][2] = {{128, 128}, {64, 128}, {128, 64}};
    static const int f64[][2] = {{64, 64}, {32, 64}, {64, 32}};
    static const int b16[][2] = {{64, 128}, {128, 128}};
    const int(*t)[2] = prec == SHTX_FP64 ? f64 : prec == SHTX_FP32 ? f32 : b16;
    int n = split_form(prec) ? 2 : 3;
    for (int i = 0; i < n && i < max; ++i) {
        bm[i] = t[i][0];
        bn[i] = t[i][1];
    }
    return n;
}

bool gemm_tile_supported(int prec, int bm, int bn)
{
    int cbm[8], cbn[8];
    int n = gemm_tile_candidates(prec, cbm, cbn, 8);
    for (int i = 0; i < n; ++i)
        if (cbm[i] == bm && cbn[i] == bn) return true;
    return false;
}

// Column fragments of the few-fields kernel for a plan and direction, 0 where
// the tiled kernels serve it.  The lines lie where the accumulators (32 FN
// registers in FP32, 64 FN in FP64) leave too few waves to cover the table's
// latency.  Microseconds against the tiled kernel: FP32 inverse, 16 fields,
// T63 8.2 / 9.2, T127 10.5 / 13.4, T255 22.6 / 23.2, T639 156 / 137, T1279 948 /
// 875 (the tiled one gains from 400 on), direct T127 10.7 / 20.9, T639 159 / 266, 32
// fields 262 / 287 (its operand loads are fewer); FP64 T639 8 fields 231 / 247 and
// 242 / 286, but 12 fields 393 / 310.
int gemm_narrow(int prec, int nfld, bool inverse)
{
    const int ncol = 2 * nfld;
    if (ncol <= 16 && (prec == SHTX_FP32 || prec == SHTX_FP64)) return 1;
    if (ncol <= 32 && prec == SHTX_FP32) return 2;
    if (ncol <= 64 && prec == SHTX_FP32 && !inverse) return 4;
    return 0;
}

bool gemm_shapes_ok(const Plan &p)
{
    const int bk = 16;
    if (!gemm_tile_supported(p.prec, p.inv_bm, p.inv_bn) || !gemm_tile_supported(p.prec, p.dir_bm, p.dir_bn))
        return false;
    // each direction's list is for its tiles, or for the few-fields kernel's
    auto dir_ok = [&](const std::vector<GemmItem> &items, bool inverse, int narrow, int bm, int bn) {
        // (one column tile holds all of that kernel's columns)
        return narrow ? 2 * p.nfld <= 16 * narrow && check_work_list(p, items, inverse, kNarrowRows, 16 * narrow, 4)
                      : check_work_list(p, items, inverse, bm, bn, bk);
    };
    return (p.inv_items.empty() || dir_ok(p.inv_items, true, p.inv_narrow, p.inv_bm, p.inv_bn)) &&
           dir_ok(p.dir_items, false, p.dir_narrow, p.dir_bm, p.dir_bn);
}

hipError_t launch_gemm_inverse(const Plan &p, const void *spec, void *four, unsigned *fmax, hipStream_t s)
{
    GemmArgs a = make_args(p, true, spec, four, false, fmax);
    if (p.inv_items.empty()) return hipSuccess;
    if (p.prec == SHTX_FP64) return launch_fp64<true>(p, a, p.inv_bm, p.inv_bn, s);
    if (p.prec == SHTX_FP32) return launch_fp32<true>(p, a, p.inv_bm, p.inv_bn, s);
    if (p.prec == SHTX_FP16X3) {
        if (!fmax) return hipErrorInvalidValue;
        k_clear_u32<<<(p.nfld + 255) / 256, 256, 0, s>>>(fmax, p.nfld);
        k_spec_absmax<<<dim3(kAbsmaxChunks, p.nfld), 1024, 0, s>>>((const float2 *)spec, p.nspec, p.trunc, fmax);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_split<SHTX_FP16X3, true>(p, a, p.inv_bm, p.inv_bn, s);
    }
    return launch_split<SHTX_BF16X3, true>(p, a, p.inv_bm, p.inv_bn, s);
}

hipError_t launch_gemm_direct(const Plan &p, const void *four, void *spec, bool adjoint, unsigned *fmax,
                              hipStream_t s)
{
    GemmArgs a = make_args(p, false, four, spec, adjoint, fmax);
    if (p.prec == SHTX_FP64) return launch_fp64<false>(p, a, p.dir_bm, p.dir_bn, s);
    if (p.prec == SHTX_FP32) return launch_fp32<false>(p, a, p.dir_bm, p.dir_bn, s);
    if (p.prec == SHTX_FP16X3) {
        // the ring r2c FFT that wrote the workspace recorded each field's maximum
        if (!fmax) return hipErrorInvalidValue;
        return launch_split<SHTX_FP16X3, false>(p, a, p.dir_bm, p.dir_bn, s);
    }
    return launch_split<SHTX_BF16X3, false>(p, a, p.dir_bm, p.dir_bn, s);
}

}  // namespace shtx
