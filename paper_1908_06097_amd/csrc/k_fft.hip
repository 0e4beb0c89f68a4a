// Batched real FFTs along the latitude rings, one launch over every
// (ring, run of fields).
//
// A real ring of n = 2h points goes through one complex DFT of length h
// (even samples as real part, odd samples as imaginary part) with the usual
// split/merge step around it.  The length-h DFT is a Stockham autosort
// mixed-radix FFT (radices up to 20 and 23; 17 in FP64) held in LDS, run in
// place: each pass reads its butterflies into registers, synchronises, then
// writes.  The first pass reads the kernel's input itself and the last writes
// its output where the radix allows.  One larger prime factor p is the first
// pass: by convolution where p - 1 has small factors and p is not small, else,
// up to 1021, a general prime pass on the matrix cores (both below); the plan's
// cost model chooses between them and Bluestein, which takes all other lengths
// through a chirp convolution at a length L = 2^a 3^b 5^c
// 7^d >= 2h - 1 chosen by the cost of its passes, with the filter spectrum
// precomputed per ring length at plan time.  Only the kept
// wavenumbers m <= M_j are read or written; they live in the Fourier
// workspace laid out [ring][m][field], so a block's loads and stores are runs
// over fields.  For the split IEEE-half Legendre form the r2c kernel also
// records each field's largest output magnitude (the bound from which the
// direct GEMM scales its data operand).
//
// Inverse (c2r):  g_k = s_j * (Re Y_0 + 2 sum_{m=1}^{M} Re(Y_m e^{2 pi i m k / n}))
//   transform:            Y_m = F_m,                    s_j = 1
//   adjoint of direct:    Y_m = F_m / c_m,              s_j = w_j / (2 n)
// Direct (r2c):   G_m = s_j fac_m sum_k g_k e^{-2 pi i m k / n},  m <= M
//   transform:            fac_m = 1,    s_j = 1 / n
//   adjoint of inverse:   fac_m = c_m,  s_j = 1
//
// The paper (Section 3.1.1) keeps fields resident on the device and packs on
// the device; this kernel's layout and algorithm are this library's own.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "fft_roots.h"
#include "shtx_internal.h"

namespace shtx {

namespace {

template <typename T>
struct __attribute__((aligned(2 * sizeof(T)))) C2 {
    T x, y;
};

template <typename T>
__device__ inline C2<T> cmul(C2<T> a, C2<T> b)
{
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ inline C2<T> cadd(C2<T> a, C2<T> b)
{
    return {a.x + b.x, a.y + b.y};
}
template <typename T>
__device__ inline C2<T> csub(C2<T> a, C2<T> b)
{
    return {a.x - b.x, a.y - b.y};
}
template <typename T>
__device__ inline C2<T> cconj(C2<T> a)
{
    return {a.x, -a.y};
}
// multiply by -i
template <typename T>
__device__ inline C2<T> cmi(C2<T> a)
{
    return {a.y, -a.x};
}

// Dynamic LDS of the FFT kernels, declared once at namespace scope so that the
// non-inlined pass functions address it as LDS (ds_* instructions) rather
// than through generic pointers.
extern __shared__ __attribute__((aligned(16))) unsigned char fft_smem[];

// Typed LDS pointers: address arithmetic on them stays 32-bit.
template <typename T>
using LdsC2 = __attribute__((address_space(3))) C2<T>;
template <typename T>
__device__ inline LdsC2<T> *lds_c2() { return (LdsC2<T> *)(__attribute__((address_space(3))) unsigned char *)fft_smem; }
// LDS byte addressing for the Stockham passes: element r of a butterfly sits
// at base + r * stride, formed with one 24-bit multiply-add per element.
typedef __attribute__((address_space(3))) unsigned char LdsByte;

// One complex value in or out of LDS as a single 2-element access.
template <typename T>
__device__ inline C2<T> ldc(const LdsC2<T> *p)
{
    typedef T V2 __attribute__((ext_vector_type(2)));
    V2 w = *(const __attribute__((address_space(3))) V2 *)p;
    return C2<T>{w.x, w.y};
}
template <typename T>
__device__ inline void stc(LdsC2<T> *p, C2<T> v)
{
    typedef T V2 __attribute__((ext_vector_type(2)));
    *(__attribute__((address_space(3))) V2 *)p = V2{v.x, v.y};
}
template <typename T>
__device__ inline C2<T> ldb(unsigned a)
{
    return ldc((const LdsC2<T> *)((LdsByte *)fft_smem + a));
}
template <typename T>
__device__ inline void stb(unsigned a, C2<T> v)
{
    stc((LdsC2<T> *)((LdsByte *)fft_smem + a), v);
}

struct FftArgs {
    const RingDesc *rings;
    const FftItem *items;
    const PassDesc *passes;
    const void *twid;
    const void *in;
    void *out;
    int nfld;
    int adjoint;
    int64_t npts;
    // r2c only, when not null: per field, the largest magnitude of the
    // Fourier values written (float bits, atomic max), collected per block in
    // nf words of LDS at byte offset fmax_lds
    unsigned *fmax;
    int fmax_lds;
};

// exp(-2 pi i t / R) for the odd prime radices (t taken mod R), as
// compile-time constants.
template <typename T, int R>
__device__ constexpr C2<T> root(int t)
{
    t %= R;
    const int u = t <= R / 2 ? t : R - t;
    const double sn = PrimeRoots<R>::s[u];
    return C2<T>{T(PrimeRoots<R>::c[u]), T(t <= R / 2 ? -sn : sn)};
}

// First of the two coprime factors of the composite radices that are formed by
// the prime-factor map (0: the radix is formed otherwise).
__host__ __device__ constexpr int pfa_factor(int R)
{
    return R == 6 || R == 10 || R == 14 || R == 18 ? 2
           : R == 12 || R == 20                   ? 4
           : R == 15                              ? 3
                                                  : 0;
}

// Forward radix-R DFT of v in registers.
template <typename T, int R>
__device__ inline void dft_reg(C2<T> *v)
{
    if constexpr (R == 2) {
        C2<T> a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (R == 3) {
        // X_1,2 = v0 - (v1 + v2)/2 -+ i (sqrt3/2)(v1 - v2)
        const T r3 = T(0.86602540378443864676372317075293618347);
        C2<T> sm = cadd(v[1], v[2]), df = csub(v[1], v[2]);
        C2<T> t = {v[0].x - T(0.5) * sm.x, v[0].y - T(0.5) * sm.y};
        C2<T> u = {r3 * df.y, -r3 * df.x};  // -i (sqrt3/2) df
        v[0] = cadd(v[0], sm);
        v[1] = cadd(t, u);
        v[2] = csub(t, u);
    } else if constexpr (R == 9) {
        // 9 = 3 x 3: radix-3 over n1 for each n2 (x = v[3 n1 + n2]), twiddles
        // exp(-2 pi i n2 k1 / 9), radix-3 over n2 for each k1
        const C2<T> tw[5] = {{T(1), T(0)},
                             {T(0.76604444311897803520239265055541667394), T(-0.64278760968653932632264340990726343291)},
                             {T(0.17364817766693034885171662676931479600), T(-0.98480775301220805936674302458952301367)},
                             {T(0), T(0)},
                             {T(-0.93969262078590838405410927732473146993), T(-0.34202014332566873304409961468225958076)}};
        C2<T> y[3][3];
#pragma unroll
        for (int n2 = 0; n2 < 3; ++n2) {
            C2<T> t[3] = {v[n2], v[3 + n2], v[6 + n2]};
            dft_reg<T, 3>(t);
#pragma unroll
            for (int k1 = 0; k1 < 3; ++k1) y[n2][k1] = (n2 && k1) ? cmul(t[k1], tw[n2 * k1]) : t[k1];
        }
#pragma unroll
        for (int k1 = 0; k1 < 3; ++k1) {
            C2<T> t[3] = {y[0][k1], y[1][k1], y[2][k1]};
            dft_reg<T, 3>(t);
#pragma unroll
            for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = t[k2];
        }
    } else if constexpr (R == 4) {
        C2<T> s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
        C2<T> s13 = cadd(v[1], v[3]), d13 = cmi(csub(v[1], v[3]));
        v[0] = cadd(s02, s13);
        v[2] = csub(s02, s13);
        v[1] = cadd(d02, d13);
        v[3] = csub(d02, d13);
    } else if constexpr (R == 8) {
        // two radix-4 DFTs (even and odd samples) merged with exp(-2 pi i k / 8)
        C2<T> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft_reg<T, 4>(e);
        dft_reg<T, 4>(o);
        const T c = T(0.70710678118654752440084436210484903928);
        C2<T> o1 = {c * (o[1].x + o[1].y), c * (o[1].y - o[1].x)};   // * (1 - i)/sqrt2
        C2<T> o2 = cmi(o[2]);                                           // * -i
        C2<T> o3 = {c * (o[3].y - o[3].x), -c * (o[3].x + o[3].y)};   // * (-1 - i)/sqrt2
        v[0] = cadd(e[0], o[0]);
        v[4] = csub(e[0], o[0]);
        v[1] = cadd(e[1], o1);
        v[5] = csub(e[1], o1);
        v[2] = cadd(e[2], o2);
        v[6] = csub(e[2], o2);
        v[3] = cadd(e[3], o3);
        v[7] = csub(e[3], o3);
    } else if constexpr (R == 16) {
        // 16 = 4 x 4: radix-4 DFTs over n1 for each n2 (x = v[4 n1 + n2]),
        // twiddles exp(-2 pi i n2 k1 / 16), radix-4 DFTs over n2 for each k1
        const T c1 = T(0.92387953251128675612818318939678828682);  // cos(pi/8)
        const T s1 = T(0.38268343236508977172845998403039886676);  // sin(pi/8)
        const T h = T(0.70710678118654752440084436210484903928);
        const C2<T> tw[10] = {{T(1), T(0)}, {c1, -s1}, {h, -h}, {s1, -c1}, {T(0), T(-1)},
                              {-s1, -c1}, {-h, -h}, {-c1, -s1}, {T(-1), T(0)}, {-c1, s1}};
        C2<T> y[4][4];
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) {
            C2<T> t[4] = {v[n2], v[4 + n2], v[8 + n2], v[12 + n2]};
            dft_reg<T, 4>(t);
#pragma unroll
            for (int k1 = 0; k1 < 4; ++k1) y[n2][k1] = (n2 && k1) ? cmul(t[k1], tw[n2 * k1]) : t[k1];
        }
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            C2<T> t[4] = {y[0][k1], y[1][k1], y[2][k1], y[3][k1]};
            dft_reg<T, 4>(t);
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = t[k2];
        }
    } else if constexpr (pfa_factor(R) > 0) {
        // R = A B with A and B coprime, by the prime-factor map: inputs
        // n = (a B + b A) mod R, A- and B-point DFTs with no twiddles between
        // them, output k at (k mod A, k mod B)
        constexpr int A = pfa_factor(R), B = R / A;
        C2<T> y[A][B];
#pragma unroll
        for (int a = 0; a < A; ++a) {
#pragma unroll
            for (int b = 0; b < B; ++b) y[a][b] = v[(a * B + b * A) % R];
            dft_reg<T, B>(y[a]);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            C2<T> t[A];
#pragma unroll
            for (int a = 0; a < A; ++a) t[a] = y[a][b];
            dft_reg<T, A>(t);
#pragma unroll
            for (int a = 0; a < A; ++a) y[a][b] = t[a];
        }
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = y[k % A][k % B];
    } else {
        // odd R: pair r with R - r
        constexpr int H = (R - 1) / 2;
        C2<T> sum[H], dif[H];
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            sum[r - 1] = cadd(v[r], v[R - r]);
            dif[r - 1] = csub(v[r], v[R - r]);
        }
        C2<T> x0 = v[0];
        C2<T> out0 = x0;
#pragma unroll
        for (int r = 0; r < H; ++r) out0 = cadd(out0, sum[r]);
#pragma unroll
        for (int k = 1; k <= H; ++k) {
            C2<T> re = x0, im = {T(0), T(0)};
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const C2<T> w = root<T, R>(k * r);  // (cos, -sin) of 2 pi k r / R
                re.x += sum[r - 1].x * w.x;
                re.y += sum[r - 1].y * w.x;
                im.x += dif[r - 1].x * w.y;
                im.y += dif[r - 1].y * w.y;
            }
            // X_k = re + i*im', X_{R-k} = re - i*im' with im' = -sum dif sin
            v[k] = {re.x - im.y, re.y + im.x};
            v[R - k] = {re.x + im.y, re.y - im.x};
        }
        v[0] = out0;
    }
}

// Elements per thread whose global loads are issued together in the
// kernels' gather and scatter loops.
constexpr int kU = 4;

// floor(a / d) as mul_hi(a, magic), magic = ceil(2^32 / d) (PassDesc): exact
// for a * d < 2^32, which every caller keeps (a and d are at most a few
// times the LDS capacity).  magic 0 stands for d = 1.
__device__ inline int udiv(int a, unsigned magic) { return magic ? (int)__umulhi((unsigned)a, magic) : a; }

// Block-uniform values passed to the non-inlined pass functions arrive in
// vector registers; these move them to scalar registers.
__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline unsigned uni(unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); }
__device__ inline PassDesc uniform(PassDesc d)
{
    d.R = uni(d.R);
    d.Ns = uni(d.Ns);
    d.nbf = uni(d.nbf);
    d.tstep = uni(d.tstep);
    d.mg_nbf = uni(d.mg_nbf);
    d.mg_ns = uni(d.mg_ns);
    return d;
}


// The table reads behind the twiddle powers of one butterfly: w = W[t1]
// (w = exp(-2 pi i k / (Ns R))) and, for radix 9, w^3, for the radices from
// 10 to 20, w^4.
template <int R>
constexpr int twiddle_step2() { return R == 9 ? 3 : R >= 10 && R != 23 ? 4 : 0; }

// Powers w^r (r = 1 .. R-1) from w and the second table value, by products
// at most three deep; tw[0] is unused.
template <typename T, int R>
__device__ inline void twiddle_powers(C2<T> *tw, C2<T> w1, C2<T> w2nd)
{
    tw[1] = w1;
    if constexpr (R == 9) {
        tw[2] = cmul(tw[1], tw[1]);
        tw[3] = w2nd;
        tw[6] = cmul(w2nd, w2nd);
#pragma unroll
        for (int a = 3; a <= 6; a += 3)
#pragma unroll
            for (int b = 1; b <= 2; ++b) tw[a + b] = cmul(tw[a], tw[b]);
    } else if constexpr (twiddle_step2<R>() == 4) {
        tw[2] = cmul(tw[1], tw[1]);
        tw[3] = cmul(tw[1], tw[2]);
        tw[4] = w2nd;
        tw[8] = cmul(w2nd, w2nd);
        if constexpr (R > 12) tw[12] = cmul(w2nd, tw[8]);
        if constexpr (R > 16) tw[16] = cmul(tw[8], tw[8]);
#pragma unroll
        for (int a = 4; a < R; a += 4)
#pragma unroll
            for (int b = 1; b <= 3; ++b)
                if (a + b < R) tw[a + b] = cmul(tw[a], tw[b]);
    } else {
        if constexpr (R > 2) tw[2] = cmul(tw[1], tw[1]);
        if constexpr (R > 3) tw[3] = cmul(tw[1], tw[2]);
        if constexpr (R > 4) tw[4] = cmul(tw[2], tw[2]);
#pragma unroll
        for (int r = 5; r < R; ++r) tw[r] = cmul(tw[4], tw[r - 4]);
    }
}

// Radix-R DFT (R odd prime) of v, written to LDS as it is formed: output t
// goes to byte address a0 + t * stride.  Sums and differences of the pairs
// (r, R - r) replace the inputs in place, so only the inputs and two
// accumulators are live (the same arithmetic as dft_reg's odd radices).
template <typename T, int R>
__device__ inline void odd_butterfly_store(C2<T> *v, unsigned a0, unsigned stride)
{
    constexpr int H = (R - 1) / 2;
    const C2<T> x0 = v[0];
    C2<T> out0 = x0;
#pragma unroll
    for (int r = 1; r <= H; ++r) {
        const C2<T> sm = cadd(v[r], v[R - r]), df = csub(v[r], v[R - r]);
        v[r] = sm;
        v[R - r] = df;
        out0 = cadd(out0, sm);
    }
    stb<T>(a0, out0);
#pragma unroll
    for (int k = 1; k <= H; ++k) {
        C2<T> re = x0, im = {T(0), T(0)};
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            const C2<T> w = root<T, R>(k * r);  // (cos, -sin) of 2 pi k r / R
            re.x += v[r].x * w.x;
            re.y += v[r].y * w.x;
            im.x += v[R - r].x * w.y;
            im.y += v[R - r].y * w.y;
        }
        stb<T>(a0 + __umul24((unsigned)k, stride), C2<T>{re.x - im.y, re.y + im.x});
        stb<T>(a0 + __umul24((unsigned)(R - k), stride), C2<T>{re.x + im.y, re.y - im.x});
    }
}

// One in-place Stockham pass of radix R over nf fields of length L in LDS:
// every thread reads all of its butterflies into registers, the block
// synchronises, then each butterfly is twiddled, transformed and written.
template <typename T>
using GlobalC2 = const __attribute__((address_space(1))) C2<T>;
template <typename T>
__device__ inline C2<T> ldg(GlobalC2<T> *p)
{
    typedef T V2 __attribute__((ext_vector_type(2)));
    const V2 w = *(const __attribute__((address_space(1))) V2 *)p;
    return C2<T>{w.x, w.y};
}

// A prime pass by convolution (C. M. Rader, Proc. IEEE 56 (1968) 1107): with g
// a primitive root of p, a length-p DFT's outputs at g^-q, but for x_0, are the
// cyclic convolution over q of its inputs at g^k with W_p^(g^-k), which two
// FFTs of length P = p - 1 make.  The pass at Ns = 1 of a ring of h = p per is
// per such transforms a field, of inputs i + r per and outputs i p + t.  Its
// passes stay in LDS: kPassGather, a Stockham pass that reads the inputs in the
// order g^k and leaves transform i at i p, entry P taking x_0; kPassSub; the
// seam of the two FFTs; kPassSub; and kPassScatter, which writes the outputs in
// the order g^-k.  Both permutations are read from memory (one table for all
// fields, in the L2).  Like Bluestein, bound by vector and LDS work, but over p
// - 1 values and not twice h: FP32, 411 fields, ps per grid point, c2r / r2c,
// against the general prime pass or Bluestein before: 2424 points (p = 101)
// 3.6 / 3.7 -> 3.2 / 3.25, 2416 (151) 4.2 / 4.15 -> 3.1 / 3.1, 1604 (401)
// 5.8 / 5.7 -> 3.7 / 3.6, 4036 (1009) 9.0 / 8.4 -> 3.6 / 3.4, 5042 (2521)
// 8.3 / 7.5 -> 4.5 / 4.4; FP64 1604 12.3 / 13.4 -> 7.4 / 8.6, 4034 (2017)
// 14.1 / 13.2 -> 7.8 / 7.8.

// Where the transforms of a pass lie in LDS: n of them, transform s at
// a s + b (s / per): the fields' slots (per = 1, b = 0), or the per = h / p
// length-p transforms of each field that a prime pass by convolution makes
// (a = p, a per + b entries a field).
struct Slots {
    int n, a, b, per;
    unsigned mg;  // div_magic(per)
};
__device__ inline Slots uniform(const Slots &s)
{
    return Slots{uni(s.n), uni(s.a), uni(s.b), uni(s.per), (unsigned)uni((int)s.mg)};
}

// Entry k of a permutation (part 0: g^k, 1: g^-k), stored as 2^23 (FP64: 2^52)
// plus the number, which is then the low bits of its low word.
template <typename T>
__device__ inline int perm_entry(GlobalC2<T> *perm, int k, int part)
{
    const unsigned w = ((const __attribute__((address_space(1))) unsigned *)(perm + (unsigned)k))[part * sizeof(T) / 4];
    return (int)(sizeof(T) == 4 ? w & 0x7fffffu : w);
}

// One pass in LDS, in place.  KIND: kPassLds over the fields' slots, and for a
// prime pass by convolution kPassGather, kPassSub and kPassScatter (below).
template <typename T, int R, int CAP, int KIND>
__device__ __attribute__((noinline)) void stockham_pass(Slots sl, PassDesc pd, GlobalC2<T> *W, GlobalC2<T> *perm)
{
    constexpr int NB = fft_rounds(CAP, R);
    constexpr int C2ND = twiddle_step2<R>();
    constexpr unsigned CB = sizeof(C2<T>);
    constexpr bool SUB = KIND != kPassLds, GATHER = KIND == kPassGather, SCATTER = KIND == kPassScatter;
    pd = uniform(pd);
    sl = uniform(sl);
    const int nbf = pd.nbf, total = sl.n * nbf, Ns = GATHER ? 1 : pd.Ns;
    const unsigned srd = nbf * CB, swr = Ns * CB;  // byte strides of a butterfly's reads and writes
    // radices above 19 run a streamed butterfly: twiddles by stepping from
    // table values read every 8 powers, outputs stored as they are formed
    constexpr bool STREAM = R > 19;
    constexpr int NRS = STREAM ? (R + 6) / 8 : 1;  // table restarts at powers 1, 9, 17, 25
    C2<T> v[NB][R];
    C2<T> w1[NB], w2[NB];  // twiddle table values, fetched before the barrier
    C2<T> wrs[NB][NRS];
    int fo[NB], qk[NB][2];
    // input 0 of the thread's transform goes to the extra entry after the
    // others, and output 0 comes from there
    C2<T> x0{};
    unsigned x0_to = 0;
    const int t0 = threadIdx.x;
    if ((GATHER || SCATTER) && t0 < sl.n) {
        const int fld = udiv(t0, sl.mg);
        const unsigned in = (unsigned)(fld * (sl.a * sl.per + sl.b) + t0 - fld * sl.per) * CB;
        const unsigned base = (unsigned)(t0 * sl.a + fld * sl.b) * CB, extra = base + (unsigned)(nbf * R) * CB;
        x0 = ldb<T>(GATHER ? in : extra);
        x0_to = GATHER ? extra : base;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        int e = threadIdx.x + b * kFftThreads;
        if (e < total) {
            int f = udiv(e, pd.mg_nbf), j = e - f * nbf;
            int q = GATHER ? j : udiv(j, pd.mg_ns), k = j - q * Ns;
            const int fld = SUB ? udiv(f, sl.mg) : 0;
            fo[b] = f * sl.a + fld * sl.b;
            qk[b][0] = q;
            qk[b][1] = k;
            if (Ns > 1) {
                const int t1 = k * pd.tstep;
                w1[b] = C2<T>{W[t1].x, W[t1].y};
                if constexpr (C2ND > 0) w2[b] = C2<T>{W[C2ND * t1].x, W[C2ND * t1].y};
                if constexpr (STREAM) {
#pragma unroll
                    for (int c = 0; c < NRS; ++c) wrs[b][c] = C2<T>{W[(8 * c + 1) * t1].x, W[(8 * c + 1) * t1].y};
                }
            }
            if constexpr (GATHER) {
                // input k of transform i of a field is entry i + g^k h / p
                const unsigned a0 = (unsigned)(fld * (sl.a * sl.per + sl.b) + f - fld * sl.per) * CB;
                int gk[R];
#pragma unroll
                for (int r = 0; r < R; ++r) gk[r] = perm_entry<T>(perm, j + r * nbf, 0);
#pragma unroll
                for (int r = 0; r < R; ++r) v[b][r] = ldb<T>(a0 + __umul24((unsigned)gk[r], (unsigned)sl.per * CB));
            } else {
                const unsigned a0 = (unsigned)(fo[b] + j) * CB;
#pragma unroll
                for (int r = 0; r < R; ++r) v[b][r] = ldb<T>(a0 + __umul24((unsigned)r, srd));
            }
        }
    }
    __syncthreads();
    if ((GATHER || SCATTER) && t0 < sl.n) stb<T>(x0_to, x0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        int e = threadIdx.x + b * kFftThreads;
        if (e < total) {
            const int q = qk[b][0], k = qk[b][1];
            int to[SCATTER ? R : 1];  // where the outputs go, fetched over the butterfly
            if constexpr (SCATTER) {
#pragma unroll
                for (int r = 0; r < R; ++r) to[r] = perm_entry<T>(perm, k + r * nbf, 1);
            }
            const int base = q * Ns * R + k;
            const unsigned a0 = (unsigned)(fo[b] + base) * CB;
            if constexpr (STREAM) {
                static_assert(!SCATTER, "streamed butterflies store at a stride");
                if (Ns > 1) {
                    C2<T> t = wrs[b][0];
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        if (r > 1) t = ((r - 1) % 8 == 0) ? wrs[b][(r - 1) / 8] : cmul(t, w1[b]);
                        v[b][r] = cmul(v[b][r], t);
                    }
                }
                odd_butterfly_store<T, R>(v[b], a0, swr);
            } else {
                if (Ns > 1) {
                    C2<T> tw[R];
                    twiddle_powers<T, R>(tw, w1[b], w2[b]);
#pragma unroll
                    for (int r = 1; r < R; ++r) v[b][r] = cmul(v[b][r], tw[r]);
                }
                dft_reg<T, R>(v[b]);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if constexpr (SCATTER)
                        stb<T>((unsigned)(fo[b] + to[r]) * CB, cconj(v[b][r]));
                    else
                        stb<T>(a0 + __umul24((unsigned)r, swr), v[b][r]);
                }
            }
        }
    }
    __syncthreads();
}

// Twiddles (for Ns > 1) and radix-R butterfly of v, from the twiddle table
// values w1 and w2 of the butterfly.
template <typename T, int R>
__device__ inline void twiddled_dft(C2<T> *v, int Ns, C2<T> w1, C2<T> w2)
{
    if (Ns > 1) {
        C2<T> tw[R];
        twiddle_powers<T, R>(tw, w1, w2);
#pragma unroll
        for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[r]);
    }
    dft_reg<T, R>(v);
}

// The seam of Bluestein's two FFTs: the first one's last pass and the second
// one's first pass have the same radix R, and then a butterfly of the one
// leaves exactly the inputs of a butterfly of the other (outputs k + t L / R,
// inputs j + t L / R), so both run in registers around the filter,
// conj(X_i bhat_i), and the two FFTs need one pass through LDS less.  Bluestein
// rings are bound by their passes' vector and LDS work (three times a plain
// ring's, at under 1 TB/s); against two whole FFTs of radix-9, -16 and smaller
// passes at the next 2^a 3^b length, 411 fields, ps per grid point, c2r / r2c:
// 5116 points 9.8 / 9.1 -> 8.1 / 7.2, 4076 11.6 / 10.7 -> 8.6 / 8.1, 2572
// 8.1 / 8.2 -> 6.0 / 5.8, 2348 9.5 / 9.5 -> 5.9 / 5.9; FP64 4996 20.0 / 17.6 ->
// 16.1 / 14.0.
//
// SUB: the seam of a prime pass by convolution, whose bin 0 is the sum of all
// inputs but x_0: with x_0 (the extra entry) it is the transform's output 0,
// kept in the extra entry, and x_0 joins every other output by bin 0.
template <typename T, int R, int CAP, bool SUB>
__device__ __attribute__((noinline)) void seam_pass(Slots sl, PassDesc pd, GlobalC2<T> *W, GlobalC2<T> *bhat)
{
    constexpr int NB = fft_rounds(CAP, R), C2ND = twiddle_step2<R>();
    constexpr unsigned CB = sizeof(C2<T>);
    pd = uniform(pd);
    sl = uniform(sl);
    const int nbf = pd.nbf, total = sl.n * nbf;
    const unsigned srd = nbf * CB;
    C2<T> v[NB][R], x0[NB];
    int fo[NB], fj[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int e = threadIdx.x + b * kFftThreads;
        if (e < total) {
            const int f = udiv(e, pd.mg_nbf), j = e - f * nbf;
            fo[b] = f * sl.a + (SUB ? udiv(f, sl.mg) * sl.b : 0);
            fj[b] = j;
            const C2<T> w1 = ldg<T>(W + (unsigned)j);
            C2<T> w2{};
            if constexpr (C2ND > 0) w2 = ldg<T>(W + (unsigned)(C2ND * j));
            const unsigned a0 = (unsigned)(fo[b] + j) * CB;
            if (SUB && j == 0) x0[b] = ldb<T>(a0 + (unsigned)(R * nbf) * CB);
#pragma unroll
            for (int r = 0; r < R; ++r) v[b][r] = ldb<T>(a0 + __umul24((unsigned)r, srd));
            twiddled_dft<T, R>(v[b], nbf, w1, w2);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // four filter values in registers at a time
                const C2<T> x = v[b][r];
                v[b][r] = cconj(cmul(x, ldg<T>(bhat + (unsigned)(j + r * nbf))));
                if (SUB && r == 0 && j == 0) {
                    v[b][0] = cadd(v[b][0], cconj(x0[b]));
                    x0[b] = cadd(x0[b], x);
                }
            }
            dft_reg<T, R>(v[b]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if ((int)threadIdx.x + b * kFftThreads >= total) continue;
        const unsigned a0 = (unsigned)(fo[b] + fj[b] * R) * CB;
#pragma unroll
        for (int r = 0; r < R; ++r) stb<T>(a0 + r * CB, v[b][r]);
        if (SUB && fj[b] == 0) stb<T>((unsigned)(fo[b] + R * nbf) * CB, x0[b]);
    }
    __syncthreads();
}

// The first and last passes of a ring's FFT join the kernels' global reads and
// writes: a pass of its own costs every value an LDS write, an LDS read, two
// barriers and the index arithmetic of a separate loop.  Measured on 64 rings
// of 5120 points (half-length 10 x 16 x 16), 411 fields: c2r 2.64 -> 2.22 and
// r2c 2.65 -> 1.99 ps per grid point; all of O1280 (most of it prime passes,
// which only the last pass helps) 12.34 -> 11.50 and 12.28 -> 11.33 ms.  What
// remains on such a ring is half memory traffic (6 bytes a point, 1.2 ps at the
// copy rate) and half vector instructions (94 per complex value).  None of
// these passes needs its butterflies held over a barrier (they read or write
// LDS, not both), so a thread takes its butterflies in runs of NB, whose loads
// are issued together.

template <typename T>
using GlobalReal = __attribute__((address_space(1))) T;
template <typename T>
using GlobalOut = __attribute__((address_space(1))) C2<T>;
template <typename T>
__device__ inline void stg(GlobalOut<T> *p, C2<T> v)
{
    typedef T V2 __attribute__((ext_vector_type(2)));
    *(__attribute__((address_space(1))) V2 *)p = V2{v.x, v.y};
}

// Values the fused passes share: the block's fields and, on the grid side,
// its first field's grid row of the ring (field f at grid + f npts) and the
// chirp of a Bluestein ring; on the Fourier side, its first field's column of
// the ring's Fourier rows ((m, f) at four[m nfld + f]) and e^{-2 pi i m / n}.
template <typename T>
struct GridSide {
    int lbufp, nf, h;
    unsigned npts;
    GlobalReal<T> *grid;
    GlobalC2<T> *chirp;
};
template <typename T>
struct FourSide {
    int lbufp, nf, h, M;
    unsigned nfld, mg_nf;
    GlobalOut<T> *four;
    GlobalC2<T> *post;
};
template <typename P>
__device__ inline P *uni(P *p)
{
    const uint64_t x = (uint64_t)(uintptr_t)p;
    return (P *)(uintptr_t)(((uint64_t)uni((unsigned)(x >> 32)) << 32) | uni((unsigned)x));
}

// First pass of the r2c FFT (Ns = 1): butterfly j of field f reads
// z_i = g_{2i} + i g_{2i+1}, i = j + r nbf, from the grid row (consecutive
// lanes take consecutive i) and writes LDS.  BLUE: times the chirp, zero for
// i >= h.
template <typename T, int R, bool BLUE>
__device__ __attribute__((noinline)) void pass_from_grid(GridSide<T> g, PassDesc pd)
{
    constexpr int NB = R >= 16 ? 1 : 16 / R;
    constexpr unsigned CB = sizeof(C2<T>);
    pd = uniform(pd);
    const int lbufp = uni(g.lbufp), nf = uni(g.nf), h = uni(g.h), nbf = pd.nbf, total = nf * nbf;
    const unsigned npts = uni(g.npts);
    GlobalReal<T> *grid = uni(g.grid);
    GlobalC2<T> *chirp = uni(g.chirp);
    for (int e0 = threadIdx.x; e0 < total; e0 += NB * kFftThreads) {
        C2<T> v[NB][R];
        int at[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int e = e0 + b * kFftThreads;
            at[b] = -1;
            if (e < total) {
                const int f = udiv(e, pd.mg_nbf), j = e - f * nbf;
                at[b] = f * lbufp + j * R;
                GlobalC2<T> *src = (GlobalC2<T> *)(grid + (uint64_t)(unsigned)f * npts);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const unsigned i = (unsigned)(j + r * nbf);
                    v[b][r] = C2<T>{T(0), T(0)};
                    if (!BLUE || i < (unsigned)h) v[b][r] = ldg<T>(src + i);
                }
                if constexpr (BLUE) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const unsigned i = (unsigned)(j + r * nbf);
                        if (i < (unsigned)h) v[b][r] = cmul(v[b][r], ldg<T>(chirp + i));
                    }
                }
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (at[b] < 0) continue;
            dft_reg<T, R>(v[b]);
            const unsigned a0 = (unsigned)at[b] * CB;
#pragma unroll
            for (int r = 0; r < R; ++r) stb<T>(a0 + r * CB, v[b][r]);
        }
    }
    __syncthreads();
}

// Last pass of the c2r FFT (Ns = nbf): z = conj(DFT), its real parts the even
// samples and its imaginary parts the odd ones, straight to the grid row.
// BLUE: the first h outputs of Bluestein's second FFT, conjugated and times
// the chirp.
template <typename T, int R, bool BLUE>
__device__ __attribute__((noinline)) void pass_to_grid(GridSide<T> g, PassDesc pd, GlobalC2<T> *W, T scale)
{
    constexpr int NB = R >= 8 || BLUE ? 1 : 8 / R;
    constexpr int C2ND = twiddle_step2<R>();
    constexpr unsigned CB = sizeof(C2<T>);
    pd = uniform(pd);
    const int lbufp = uni(g.lbufp), nf = uni(g.nf), h = uni(g.h), nbf = pd.nbf, total = nf * nbf;
    const unsigned npts = uni(g.npts), srd = nbf * CB;
    GlobalReal<T> *grid = uni(g.grid);
    GlobalC2<T> *chirp = uni(g.chirp);
    for (int e0 = threadIdx.x; e0 < total; e0 += NB * kFftThreads) {
        C2<T> v[NB][R], w1[NB], w2[NB];
        int ff[NB], jj[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int e = e0 + b * kFftThreads;
            ff[b] = -1;
            if (e < total) {
                const int f = udiv(e, pd.mg_nbf), j = e - f * nbf;
                ff[b] = f;
                jj[b] = j;
                if (nbf > 1) {
                    w1[b] = ldg<T>(W + (unsigned)j);
                    if constexpr (C2ND > 0) w2[b] = ldg<T>(W + (unsigned)(C2ND * j));
                }
                const unsigned a0 = (unsigned)(f * lbufp + j) * CB;
#pragma unroll
                for (int r = 0; r < R; ++r) v[b][r] = ldb<T>(a0 + __umul24((unsigned)r, srd));
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (ff[b] < 0) continue;
            twiddled_dft<T, R>(v[b], nbf, w1[b], w2[b]);
            GlobalOut<T> *dst = (GlobalOut<T> *)(grid + (uint64_t)(unsigned)ff[b] * npts);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned i = (unsigned)(jj[b] + r * nbf);
                if constexpr (BLUE) {
                    // four chirp values in registers at a time
                    if (r % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                    if (i < (unsigned)h) {
                        const C2<T> z = cmul(ldg<T>(chirp + i), cconj(v[b][r]));
                        stg<T>(dst + i, C2<T>{scale * z.x, -scale * z.y});
                    }
                } else {
                    stg<T>(dst + i, C2<T>{scale * v[b][r].x, -scale * v[b][r].y});
                }
            }
        }
    }
}

// Merge step of the c2r transform for the pair (m, h - m): from y0 = Y_m and
// y1 = Y_{h-m} (the latter zero for m = 0) and pst = e^{-2 pi i m / n},
//   Z'_m = (Y_m + conj Y_{h-m}) + i e^{2 pi i m / n} (Y_m - conj Y_{h-m})
// and its mirror; y0 and y1 become conj Z'_m and conj Z'_{h-m}.
template <typename T>
__device__ inline void merge_pair(C2<T> &y0, C2<T> &y1, C2<T> pst)
{
    const C2<T> A = {y0.x + y1.x, y0.y - y1.y}, B = {y0.x - y1.x, y0.y + y1.y};
    const C2<T> t = cmul(cconj(pst), B);
    y0 = {A.x - t.y, -A.y - t.x};
    y1 = {A.x + t.y, A.y - t.x};
}

// Y_m / 2 of the adjoint of the direct transform, m > 0.  (Y_0 doubled and the
// half in the last scale is one multiplication less, but overflows for F_0 from
// half the largest value on.)
template <typename T>
__device__ inline C2<T> halved(C2<T> y)
{
    return {T(0.5) * y.x, T(0.5) * y.y};
}

// First pass of the c2r FFT (Ns = 1) with the merge step: a thread takes the
// butterflies u and nbf - u of one field, whose inputs are each other's
// mirrors (h - (u + r nbf) = (nbf - u) + (R - 1 - r) nbf), so that every
// Fourier value is read once and merged in registers.  Consecutive lanes take
// consecutive fields of a row (the runs in memory).  adjoint: Y_m = F_m / c_m.
template <typename T, int R>
__device__ __attribute__((noinline)) void pass_from_four(FourSide<T> g, PassDesc pd, bool adjoint)
{
    constexpr int NB = R >= 8 ? 1 : 8 / R;
    constexpr unsigned CB = sizeof(C2<T>);
    pd = uniform(pd);
    const int lbufp = uni(g.lbufp), nf = uni(g.nf), M = uni(g.M), nbf = pd.nbf, total = nf * (nbf / 2 + 1);
    const unsigned nfld = uni(g.nfld), mg_nf = uni(g.mg_nf);
    GlobalC2<T> *four = (GlobalC2<T> *)uni(g.four), *post = uni(g.post);
    for (int e0 = threadIdx.x; e0 < total; e0 += NB * kFftThreads) {
        C2<T> ya[NB][R], yb[NB][R], ps[NB][R];
        int uu[NB], ff[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int e = e0 + b * kFftThreads;
            uu[b] = -1;
            if (e < total) {
                const int u = udiv(e, mg_nf), f = e - u * nf;
                uu[b] = u;
                ff[b] = f;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int m = u + r * nbf, q = nbf - u + r * nbf;
                    ya[b][r] = C2<T>{T(0), T(0)};
                    yb[b][r] = C2<T>{T(0), T(0)};
                    if (m <= M) ya[b][r] = ldg<T>(four + ((unsigned)m * nfld + (unsigned)f));
                    if (q <= M) yb[b][r] = ldg<T>(four + ((unsigned)q * nfld + (unsigned)f));
                    ps[b][r] = ldg<T>(post + (unsigned)m);
                }
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int u = uu[b];
            if (u < 0) continue;
            if (u == 0) ya[b][0].y = T(0);
            if (adjoint) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (u + r > 0) ya[b][r] = halved(ya[b][r]);
                    yb[b][r] = halved(yb[b][r]);
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) merge_pair(ya[b][r], yb[b][R - 1 - r], ps[b][r]);
            dft_reg<T, R>(ya[b]);
            const unsigned a0 = (unsigned)(ff[b] * lbufp + u * R) * CB;
#pragma unroll
            for (int r = 0; r < R; ++r) stb<T>(a0 + r * CB, ya[b][r]);
            if (u > 0 && 2 * u < nbf) {
                dft_reg<T, R>(yb[b]);
                const unsigned a1 = (unsigned)(ff[b] * lbufp + (nbf - u) * R) * CB;
#pragma unroll
                for (int r = 0; r < R; ++r) stb<T>(a1 + r * CB, yb[b][r]);
            }
        }
    }
    __syncthreads();
}

// One Fourier value of the r2c transform to its row, and its magnitude to the
// field's maximum (smax: LDS words per field, or null).
typedef __attribute__((address_space(3))) unsigned LdsWord;
template <typename T>
__device__ inline void put_four(GlobalOut<T> *four, unsigned nfld, int m, int f, C2<T> y, LdsWord *smax)
{
    stg<T>(four + ((unsigned)m * nfld + (unsigned)f), y);
    if (smax)
        __hip_atomic_fetch_max(smax + f, __float_as_uint((float)fmax(fabs(y.x), fabs(y.y))), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Last pass of the r2c FFT (Ns = nbf) with the split step
//   Y_m = (Z_m + conj Z_{h-m}) / 2 - (i/2) e^{-2 pi i m / n} (Z_m - conj Z_{h-m}):
// a thread takes the butterflies k and nbf - k of one field, whose outputs
// are each other's mirrors, and writes the kept Y_m (m <= M) to the Fourier
// rows.  scale0 / scale: half the transform's factor at m = 0 / m > 0.
template <typename T, int R>
__device__ __attribute__((noinline)) void pass_to_four(FourSide<T> g, PassDesc pd, GlobalC2<T> *W, T scale0, T scale,
                                                       LdsWord *smax)
{
    constexpr int C2ND = twiddle_step2<R>();
    constexpr unsigned CB = sizeof(C2<T>);
    pd = uniform(pd);
    const int lbufp = uni(g.lbufp), nf = uni(g.nf), M = uni(g.M), h = uni(g.h), nbf = pd.nbf,
              total = nf * (nbf / 2 + 1);
    const unsigned nfld = uni(g.nfld), mg_nf = uni(g.mg_nf), srd = nbf * CB;
    GlobalOut<T> *four = uni(g.four);
    GlobalC2<T> *post = uni(g.post);
    for (int e = threadIdx.x; e < total; e += kFftThreads) {
        const int k = udiv(e, mg_nf), f = e - k * nf, kb = k ? nbf - k : 0;
        C2<T> va[R], vb[R], ps[R], wa{}, wa2{}, wb{}, wb2{};
        if (nbf > 1) {
            wa = ldg<T>(W + (unsigned)k);
            wb = ldg<T>(W + (unsigned)kb);
            if constexpr (C2ND > 0) {
                wa2 = ldg<T>(W + (unsigned)(C2ND * k));
                wb2 = ldg<T>(W + (unsigned)(C2ND * kb));
            }
        }
        const unsigned a0 = (unsigned)(f * lbufp + k) * CB, a1 = (unsigned)(f * lbufp + kb) * CB;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            va[r] = ldb<T>(a0 + __umul24((unsigned)r, srd));
            vb[r] = ldb<T>(a1 + __umul24((unsigned)r, srd));
        }
        twiddled_dft<T, R>(va, nbf, wa, wa2);
        __builtin_amdgcn_sched_barrier(0);  // one butterfly's twiddles in registers at a time
        twiddled_dft<T, R>(vb, nbf, wb, wb2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < R; ++r) ps[r] = ldg<T>(post + (unsigned)(k + r * nbf));
        // k = 0 mirrors itself: Z_{h - t nbf} = Z_{(R - t) nbf}
        if (k == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) vb[r] = va[(r + 1) % R];
        }
        const bool mirror = k > 0 && 2 * k < nbf;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int m = k + r * nbf;
            const C2<T> zm = va[r], zq = vb[R - 1 - r];
            const C2<T> A = {zm.x + zq.x, zm.y - zq.y}, B = {zm.x - zq.x, zm.y + zq.y};
            const C2<T> t = cmul(ps[r], B);
            const T s = m == 0 ? scale0 : scale;
            if (m <= M) put_four<T>(four, nfld, m, f, C2<T>{s * (A.x + t.y), m == 0 ? T(0) : s * (A.y - t.x)}, smax);
            if (mirror && h - m <= M)
                put_four<T>(four, nfld, h - m, f, C2<T>{s * (A.x - t.y), s * (-A.y - t.x)}, smax);
        }
    }
}

// General prime pass (radix p = pd.R, an odd prime, first pass so Ns = 1 and
// no input twiddles), as matrix products on the matrix cores.  With x_r the
// inputs of butterfly b, w = e^{-2 pi i / p}, H = (p - 1) / 2,
//   X_t = x_0 + P_t + i Q_t,   X_{p-t} = x_0 + P_t - i Q_t,   t = 0 .. H,
//   P_t = sum_{r=1}^{H} Re(w^{rt}) s_r,   Q_t = sum_{r=1}^{H} Im(w^{rt}) d_r,
// s_r = x_r + x_{p-r}, d_r = x_r - x_{p-r}: two real products of an H x H
// matrix (cosines, sines) with an H x (2 x butterflies) matrix whose columns
// are the real and imaginary parts of s or d.  A wave computes a tile of NI x NJ
// output units of 16 x 16 (rows t, columns (butterfly, re|im)) with 16x16x4
// MFMAs: the matrix operand is read from a table of the p-th roots in LDS at
// index r t mod p, once for the NJ units of a row; the data operand forms s
// and d from the ring's LDS slots as it is read, once for the NI units of a
// column: the root reads' bank conflicts made LDS, not the matrix cores, the
// bound when each unit read its own.  64 rings of 5136 points (p = 107), 411
// fields: c2r 3.92 -> 3.54, r2c 4.16 -> 3.72 ps per grid point; 1284 points (p
// = 107) 3.70 -> 3.23; FP64 5136 points 8.7 -> 7.6.
// The units' results stay in registers over a barrier (the pass is in place);
// X_t of butterfly j then goes to j p + t.
typedef float gp_f32x4 __attribute__((ext_vector_type(4)));
typedef double gp_f64x4 __attribute__((ext_vector_type(4)));
__device__ inline gp_f32x4 gp_mfma(float a, float b, gp_f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ inline gp_f64x4 gp_mfma(double a, double b, gp_f64x4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Absolute LDS addresses (the dynamic LDS base already added), for loops that
// step addresses instead of re-adding the base at every access.
__device__ inline unsigned lds_base() { return (unsigned)(uintptr_t)(LdsByte *)fft_smem; }
template <typename T>
__device__ inline T lda(unsigned a)
{
    return *(const __attribute__((address_space(3))) T *)(uintptr_t)a;
}
// One real value to LDS at byte offset a of the dynamic LDS.
template <typename T>
__device__ inline void str(unsigned a, T v)
{
    *(__attribute__((address_space(3))) T *)((LdsByte *)fft_smem + a) = v;
}

// Geometry of a general prime pass shared by its units (block-uniform values
// and the lane's position in the 16 x 16 MFMA layout).
struct GpGeom {
    int p, H, mt, nb, nbf;
    unsigned mg_nbf;
    int lbufp, ksteps;
    unsigned rb, rstr, rspan, rstep, lb;
    int lr, lk;
};

// K loop of a wave's NI x NJ output units: for row tile i the lane's matrix
// operand row is t = 16 (i0 + i) + lr with roots w^{r t}, r = 1 + lk + 4 k,
// addressed by (r t mod p) rstr and stepped by 4 t mod p with an unsigned
// min(x, x - span) wrap; for column tile j its data operand column is
// c = 16 (g0 + j) + lr = 2 b + (re|im), forming s_r and d_r from x_r and
// x_{p-r}.  Operands of step k + 1 are read before the products of step k.
// Rows r past H in the last step contribute 0.
template <typename T, int NI, int NJ, typename V4>
__device__ __attribute__((always_inline)) inline void gp_run(const GpGeom &g, int i0, int g0, V4 (&P)[NI][NJ],
                                                             V4 (&Q)[NI][NJ], T (&x0)[NJ])
{
    constexpr unsigned CB = sizeof(C2<T>), RB = sizeof(T);
    unsigned ur[NI], du[NI], ar[NJ], am[NJ];
    C2<T> w[NI];
    T xr[NJ], xm[NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int t = 16 * (i0 + i) + g.lr;
        ur[i] = (unsigned)((t * (1 + g.lk)) % g.p) * g.rstr;
        du[i] = (unsigned)((4 * t) % g.p) * g.rstr;
        w[i] = ldc<T>((const LdsC2<T> *)(uintptr_t)(g.rb + ur[i]));
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = 16 * (g0 + j) + g.lr;
        const int b = min(c >> 1, g.nb - 1);
        const int f = udiv(b, g.mg_nbf), jj = b - f * g.nbf;
        const unsigned slot = g.lb + (unsigned)(f * g.lbufp + jj) * CB + (unsigned)(c & 1) * RB;
        ar[j] = slot + (unsigned)(1 + g.lk) * g.nbf * CB;
        am[j] = slot + (unsigned)(g.p - 1 - g.lk) * g.nbf * CB;
        x0[j] = lda<T>(slot);
        xr[j] = lda<T>(ar[j]);
        xm[j] = lda<T>(am[j]);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            P[i][j] = V4{T(0), T(0), T(0), T(0)};
            Q[i][j] = V4{T(0), T(0), T(0), T(0)};
        }
    }
    for (int k = 0; k < g.ksteps - 1; ++k) {
        C2<T> w1[NI];
        T xr1[NJ], xm1[NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const unsigned nx = ur[i] + du[i];
            ur[i] = min(nx, nx - g.rspan);
            w1[i] = ldc<T>((const LdsC2<T> *)(uintptr_t)(g.rb + ur[i]));
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            ar[j] += g.rstep;
            am[j] -= g.rstep;
            xr1[j] = lda<T>(ar[j]);
            xm1[j] = lda<T>(am[j]);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const T sm = xr[j] + xm[j], df = xr[j] - xm[j];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                P[i][j] = gp_mfma(w[i].x, sm, P[i][j]);
                Q[i][j] = gp_mfma(w[i].y, df, Q[i][j]);
            }
            xr[j] = xr1[j];
            xm[j] = xm1[j];
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) w[i] = w1[i];
    }
    const bool live = 4 * (g.ksteps - 1) + 1 + g.lk <= g.H;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const T sm = live ? xr[j] + xm[j] : T(0), df = live ? xr[j] - xm[j] : T(0);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            P[i][j] = gp_mfma(w[i].x, sm, P[i][j]);
            Q[i][j] = gp_mfma(w[i].y, df, Q[i][j]);
        }
    }
}

// The pass in tiles of NI x NJ units, one per wave (GpShape; the plan's field
// blocking leaves at most one).
template <typename T, int NI, int NJ>
__device__ __attribute__((noinline)) void gp_pass(int lbufp, int nf, PassDesc pd, GlobalC2<T> *Wg)
{
    using V4 = typename std::conditional<sizeof(T) == 4, gp_f32x4, gp_f64x4>::type;
    constexpr unsigned CB = sizeof(C2<T>), RB = sizeof(T);
    pd = uniform(pd);
    lbufp = uni(lbufp);
    nf = uni(nf);
    const int p = pd.R, H = (p - 1) / 2, nbf = pd.nbf, nb = nf * nbf;
    const int mt = gp_row_tiles(p), ct = gp_col_tiles(nb), ksteps = (H + 3) / 4;
    // 1. w^u = W_L[u nbf] (u < p) to a table of p roots after the field slots
    const int roots_off = nf * lbufp;
    for (int u = threadIdx.x; u < p; u += kFftThreads)
        stb<T>((unsigned)(roots_off + u) * CB, C2<T>{Wg[u * nbf].x, Wg[u * nbf].y});
    __syncthreads();
    const unsigned rstr = CB, rspan = (unsigned)p * rstr, rstep = 4u * nbf * CB;
    const unsigned lb = lds_base(), rb = lb + (unsigned)roots_off * CB;
    const int wave = uni((int)(threadIdx.x / 64)), lane = threadIdx.x % 64, lr = lane & 15, lk = lane >> 4;
    V4 accp[NI][NJ], accq[NI][NJ];
    T x0[NJ];
    // 2. the wave's row tiles i0 .. and column tiles g0 ..
    const GpGeom gm{p, H, mt, nb, nbf, pd.mg_nbf, lbufp, ksteps, rb, rstr, rspan, rstep, lb, lr, lk};
    const int mi = (mt + NI - 1) / NI, i0 = wave % mi * NI, g0 = wave / mi * NJ;
    if (g0 < ct) gp_run<T, NI, NJ>(gm, i0, g0, accp, accq, x0);
    __syncthreads();
    // 3. lane (column c, four rows) holds P and Q of one real component; i Q
    //    takes the other component's Q from the neighbour lane.  Output rows of
    //    the 16x16x4 MFMA: 4 (lane / 16) + v in FP32, lane / 16 + 4 v in FP64.
    if (g0 < ct) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int c = 16 * (g0 + j) + lr, b = c >> 1, im = c & 1;
            const int f = udiv(min(b, nb - 1), pd.mg_nbf), jj = min(b, nb - 1) - f * nbf;
            const unsigned ob = (unsigned)(f * lbufp + jj * p) * CB + (unsigned)im * RB;
            const T sg = im ? T(1) : T(-1);
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const T qo = __shfl_xor(accq[i][j][v], 1);
                    const int t = 16 * (i0 + i) + (sizeof(T) == 8 ? lk + 4 * v : 4 * lk + v);
                    if (b < nb && t <= H) {
                        str<T>(ob + (unsigned)t * CB, x0[j] + accp[i][j][v] + sg * qo);
                        if (t > 0) str<T>(ob + (unsigned)(p - t) * CB, x0[j] + accp[i][j][v] - sg * qo);
                    }
                }
        }
    }
    __syncthreads();
}

// The prime pass in the tile shape of the work item.
template <typename T>
__device__ inline void gp_dispatch(int shape, int lbufp, int nf, const PassDesc &pd, GlobalC2<T> *W)
{
#define SHTX_GP(NI, NJ)                                                                 \
    case gp_shape(NI, NJ):                                                              \
        gp_pass<T, NI, NJ>(lbufp, nf, pd, W);                                           \
        break;
    switch (shape) {
        SHTX_GP_SHAPES(SHTX_GP)
    }
#undef SHTX_GP
}

// Calls fn(std::integral_constant<int, R>) for the radix R of a pass of one
// kind (the plan checks hold every pass to fft_radix_ok).
template <int KIND, bool DBL, typename Fn>
__device__ inline void radix_dispatch(int R, Fn fn)
{
#define SHTX_RADIX(X)                                                             \
    case X:                                                                       \
        if constexpr (fft_radix_ok(KIND, DBL, X)) fn(std::integral_constant<int, X>{}); \
        break;
    switch (R) {
        SHTX_RADIX(2)
        SHTX_RADIX(3)
        SHTX_RADIX(4)
        SHTX_RADIX(5)
        SHTX_RADIX(6)
        SHTX_RADIX(7)
        SHTX_RADIX(8)
        SHTX_RADIX(9)
        SHTX_RADIX(10)
        SHTX_RADIX(11)
        SHTX_RADIX(12)
        SHTX_RADIX(13)
        SHTX_RADIX(14)
        SHTX_RADIX(15)
        SHTX_RADIX(16)
        SHTX_RADIX(17)
        SHTX_RADIX(18)
        SHTX_RADIX(19)
        SHTX_RADIX(20)
        SHTX_RADIX(23)
    }
#undef SHTX_RADIX
}

template <typename T, int CAP>
__device__ inline void pass_dispatch(int lbufp, int nf, int shape, const PassDesc &pd, const C2<T> *W)
{
    if (gp_radix(pd.R, sizeof(T) == 8)) {
        gp_dispatch<T>(shape, lbufp, nf, pd, (GlobalC2<T> *)W);
        return;
    }
    radix_dispatch<kPassLds, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
        stockham_pass<T, decltype(r)::value, CAP, kPassLds>(Slots{nf, lbufp, 0, 1, 0u}, pd, (GlobalC2<T> *)W, nullptr);
    });
}

// One pass of a prime pass by convolution.
template <typename T, int CAP, int KIND>
__device__ inline void sub_dispatch(const Slots &sl, const PassDesc &pd, const C2<T> *W, const C2<T> *perm)
{
    radix_dispatch<KIND, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
        stockham_pass<T, decltype(r)::value, CAP, KIND>(sl, pd, (GlobalC2<T> *)W, (GlobalC2<T> *)perm);
    });
}

// Passes first .. last - 1 of each field slot's FFT; pass `seam` (Bluestein; -1:
// none) is the seam of its two FFTs: the input must already be multiplied by
// the chirp and zero-padded to L, the second FFT leaves conj(conv), and the
// caller multiplies by the chirp when reading the first h outputs.
template <typename T, int CAP>
__device__ inline void dft_passes(const RingDesc &d, const PassDesc *ps, int seam, int first, int last, int nf,
                                  int shape, const C2<T> *tw)
{
    const C2<T> *W = tw + d.tw_off, *bhat = tw + d.bhat_off;
    if (d.conv) {
        const C2<T> *Wp = tw + d.conv_tw_off, *perm = tw + d.conv_perm_off;
        const int per = uni(d.h) / uni(d.conv_p);
        const Slots sl{nf * per, d.conv_p, d.lbufp - d.h, per, div_magic(per)};
        for (int s = 0; s < d.conv; ++s) {
            const PassDesc pd = ps[s];
            if (s == 0)
                sub_dispatch<T, CAP, kPassGather>(sl, pd, Wp, perm);
            else if (s == seam)
                radix_dispatch<kPassSubSeam, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
                    seam_pass<T, decltype(r)::value, CAP, true>(sl, pd, (GlobalC2<T> *)Wp, (GlobalC2<T> *)bhat);
                });
            else if (s == d.conv - 1)
                sub_dispatch<T, CAP, kPassScatter>(sl, pd, Wp, perm);
            else
                sub_dispatch<T, CAP, kPassSub>(sl, pd, Wp, nullptr);
        }
        first = d.conv;
        seam = -1;
    }
    for (int s = first; s < last; ++s) {
        const PassDesc pd = ps[s];
        if (s == seam)
            radix_dispatch<kPassSeam, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
                seam_pass<T, decltype(r)::value, CAP, false>(Slots{nf, d.lbufp, 0, 1, 0u}, pd, (GlobalC2<T> *)W,
                                                             (GlobalC2<T> *)bhat);
            });
        else
            pass_dispatch<T, CAP>(d.lbufp, nf, shape, pd, W);
    }
}

// A ring's grid rows can be moved two complex values (four points) at a time
// with 16-byte accesses: no chirp, even h, and every field's row of the ring
// starting on a 16-byte boundary (the block's first row aligned, field stride
// a multiple of 4 points).
__device__ inline bool grid_pairs(const RingDesc &d, int h, unsigned npts, const void *row0)
{
    return !d.blue && (h & 1) == 0 && (npts & 3u) == 0 && (reinterpret_cast<uintptr_t>(row0) & 15) == 0;
}

// The c2r kernel's reads of the kept coefficients Y_m, Y_{h-m} (m <= M) where
// its first pass does not take them itself (general prime passes, Bluestein):
// merged into u = conj(Z') in LDS, for Bluestein times the chirp and
// zero-padded to L.  Runs over fields are contiguous in memory; each thread
// issues the loads of kU elements before using any.
template <typename T>
__device__ inline void merge_to_lds(const RingDesc &d, const C2<T> *fourb, unsigned nfld, int nf, unsigned mg_nf,
                                    const C2<T> *post, const C2<T> *chirp, bool adjoint)
{
    LdsC2<T> *buf = lds_c2<T>();
    const int h = d.h, M = d.M, lbufp = d.lbufp;
    const int hp = h / 2 + 1, nmerge = nf * hp;
    for (int e0 = threadIdx.x; e0 < nmerge; e0 += kU * kFftThreads) {
        C2<T> ym[kU], yh[kU], pm[kU], cm[kU];
        int mm[kU], ff[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + u * kFftThreads;
            const bool ok = e < nmerge;
            int m = ok ? udiv(e, mg_nf) : 0;
            int f = ok ? e - m * nf : 0;
            mm[u] = ok ? m : -1;
            ff[u] = f;
            const C2<T> zero = {T(0), T(0)};
            ym[u] = zero;
            yh[u] = zero;
            // 32-bit unsigned element offsets from the block's base pointers
            if (ok && m <= M) ym[u] = fourb[(unsigned)m * nfld + (unsigned)f];
            if (ok && h - m <= M) yh[u] = fourb[(unsigned)(h - m) * nfld + (unsigned)f];
            pm[u] = post[(unsigned)m];
            cm[u] = zero;
            if (d.blue) cm[u] = chirp[(unsigned)m];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int m = mm[u];
            if (m < 0) continue;
            C2<T> y0 = ym[u], y1 = yh[u];
            if (m == 0) y0.y = T(0);
            if (adjoint) {
                if (m > 0) y0 = halved(y0);
                y1 = halved(y1);
            }
            merge_pair(y0, y1, pm[u]);
            if (d.blue) {
                // the chirp at h - m is the chirp at m times (-1)^h (m > 0)
                y0 = cmul(y0, cm[u]);
                y1 = cmul(y1, (h & 1) ? C2<T>{-cm[u].x, -cm[u].y} : cm[u]);
            }
            LdsC2<T> *sl = buf + ff[u] * lbufp;
            if (m != 0 && m != h - m) stc(sl + (h - m), y1);
            stc(sl + m, y0);
        }
    }
    if (d.blue) {
        const int zl = d.L - h;
        const unsigned mg_z = div_magic(zl);
        for (int e = threadIdx.x; e < nf * zl; e += kFftThreads) {
            int f = udiv(e, mg_z), k = h + e - f * zl;
            stc(buf + f * lbufp + k, C2<T>{T(0), T(0)});
        }
    }
    __syncthreads();
}

template <typename T, int CAP>
__global__ __launch_bounds__(kFftThreads, sizeof(T) == 4 ? 4 : 2) void k_fft_c2r(FftArgs a)
{
    LdsC2<T> *buf = lds_c2<T>();
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const FftItem it = a.items[item];
    if (it.ring < 0) return;
    const RingDesc d = a.rings[it.ring];
    const C2<T> *tw = (const C2<T> *)a.twid;
    const C2<T> *W = tw + d.tw_off;
    const C2<T> *post = tw + d.post_off;
    const C2<T> *chirp = tw + d.chirp_off;
    const int nf = it.nf, f0 = it.f0, h = d.h, M = d.M, lbufp = d.lbufp;
    const unsigned nfld = (unsigned)a.nfld, npts = (unsigned)a.npts;
    const C2<T> *fourb = (const C2<T> *)a.in + d.four_off + f0;  // (m, f) at fourb[m nfld + f]
    T *gridb = (T *)a.out + (uint64_t)f0 * npts + d.grid_off;    // field f at gridb + f npts
    const unsigned mg_nf = div_magic(nf);
    const bool adjoint = a.adjoint != 0;
    const T scale = adjoint ? T(d.w / (2.0 * d.n)) : T(1);
    const PassDesc *ps = a.passes + d.pass_off;
    if (d.fuse_in) {
        const FourSide<T> fs{lbufp, nf, h, M, nfld, mg_nf, (GlobalOut<T> *)fourb, (GlobalC2<T> *)post};
        const PassDesc pd = ps[0];
        radix_dispatch<kPassFromFour, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
            pass_from_four<T, decltype(r)::value>(fs, pd, adjoint);
        });
    } else {
        merge_to_lds<T>(d, fourb, nfld, nf, mg_nf, post, chirp, adjoint);
    }
    // forward DFT of length h; z = conj(DFT(u)): even samples Re z, odd samples Im z
    dft_passes<T, CAP>(d, ps, d.seam, d.fuse_in, d.nrad - d.fuse_out, nf, it.shape, tw);
    if (d.fuse_out) {
        const GridSide<T> gs{lbufp, nf, h, npts, (GlobalReal<T> *)gridb, (GlobalC2<T> *)chirp};
        const PassDesc pd = ps[d.nrad - 1];
        radix_dispatch<kPassToGrid, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
            constexpr int R = decltype(r)::value;
            if constexpr (blue_last_radix(R, sizeof(T) == 8)) {
                if (d.blue) return pass_to_grid<T, R, true>(gs, pd, (GlobalC2<T> *)W, scale);
            }
            pass_to_grid<T, R, false>(gs, pd, (GlobalC2<T> *)W, scale);
        });
        return;
    }

    // single precision, no chirp, even h and 16-byte aligned rows: two complex
    // values (four grid points) per element with one 16-byte store
    if (sizeof(T) == 4 && grid_pairs(d, h, npts, gridb)) {
        typedef T V4 __attribute__((ext_vector_type(4)));
        const int hh = h / 2;
        const unsigned mg_hh = div_magic(hh);
        for (int e0 = threadIdx.x; e0 < nf * hh; e0 += kU * kFftThreads) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = e0 + u * kFftThreads;
                if (e >= nf * hh) continue;
                const int f = udiv(e, mg_hh), kk = e - f * hh;
                const C2<T> x0 = ldc(buf + f * lbufp + 2 * kk), x1 = ldc(buf + f * lbufp + 2 * kk + 1);
                *reinterpret_cast<V4 *>(gridb + (uint64_t)(unsigned)f * npts + 4u * (unsigned)kk) =
                    V4{scale * x0.x, -scale * x0.y, scale * x1.x, -scale * x1.y};
            }
        }
        return;
    }
    const unsigned mg_h = div_magic(h);
    for (int e0 = threadIdx.x; e0 < nf * h; e0 += kU * kFftThreads) {
        C2<T> cp[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + u * kFftThreads;
            const int k = e < nf * h ? e - udiv(e, mg_h) * h : 0;
            cp[u] = d.blue ? chirp[(unsigned)k] : C2<T>{T(1), T(0)};
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + u * kFftThreads;
            if (e >= nf * h) continue;
            const int f = udiv(e, mg_h), k = e - f * h;
            const C2<T> x = ldc(buf + f * lbufp + k);
            const C2<T> r = d.blue ? cmul(cp[u], cconj(x)) : x;
            const C2<T> g = {scale * r.x, -scale * r.y};
            *reinterpret_cast<C2<T> *>(gridb + (uint64_t)(unsigned)f * npts + 2u * (unsigned)k) = g;
        }
    }
}

template <typename T, int CAP>
__global__ __launch_bounds__(kFftThreads, sizeof(T) == 4 ? 4 : 2) void k_fft_r2c(FftArgs a)
{
    LdsC2<T> *buf = lds_c2<T>();
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const FftItem it = a.items[item];
    if (it.ring < 0) return;
    const RingDesc d = a.rings[it.ring];
    const C2<T> *tw = (const C2<T> *)a.twid;
    const C2<T> *W = tw + d.tw_off;
    const C2<T> *post = tw + d.post_off;
    const C2<T> *chirp = tw + d.chirp_off;
    const int nf = it.nf, f0 = it.f0, h = d.h, M = d.M, lbufp = d.lbufp;
    const unsigned npts = (unsigned)a.npts;
    const T *gridb = (const T *)a.in + (uint64_t)f0 * npts + d.grid_off;  // field f at gridb + f npts
    LdsWord *smax = a.fmax ? (LdsWord *)((LdsByte *)fft_smem + a.fmax_lds) : nullptr;
    if (a.fmax)
        for (int f = threadIdx.x; f < nf; f += kFftThreads) smax[f] = 0u;  // ordered by the first pass's barrier

    // 1. z_k = g_{2k} + i g_{2k+1}; Bluestein: times the chirp, zero-padded to L
    const PassDesc *ps = a.passes + d.pass_off_r;
    if (d.fuse_in_r) {
        const GridSide<T> gs{lbufp, nf, h, npts, (GlobalReal<T> *)gridb, (GlobalC2<T> *)chirp};
        const PassDesc pd = ps[0];
        radix_dispatch<kPassFromGrid, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
            constexpr int R = decltype(r)::value;
            if constexpr (blue_first_radix(R, sizeof(T) == 8)) {
                if (d.blue) return pass_from_grid<T, R, true>(gs, pd);
            }
            pass_from_grid<T, R, false>(gs, pd);
        });
    }
    const int span = d.blue ? d.L : h;
    const unsigned mg_span = div_magic(span);
    // single precision, no chirp, even h and 16-byte aligned rows: four grid
    // points (two complex values) per element with one 16-byte load
    const bool pairs = sizeof(T) == 4 && grid_pairs(d, h, npts, gridb);
    if (!d.fuse_in_r && pairs) {
        typedef T V4 __attribute__((ext_vector_type(4)));
        const int hh = h / 2;
        const unsigned mg_hh = div_magic(hh);
        for (int e0 = threadIdx.x; e0 < nf * hh; e0 += kU * kFftThreads) {
            V4 gv[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = e0 + u * kFftThreads;
                if (e < nf * hh) {
                    const int f = udiv(e, mg_hh), kk = e - f * hh;
                    gv[u] = *reinterpret_cast<const V4 *>(gridb + (uint64_t)(unsigned)f * npts + 4u * (unsigned)kk);
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = e0 + u * kFftThreads;
                if (e >= nf * hh) continue;
                const int f = udiv(e, mg_hh), kk = e - f * hh;
                stc(buf + f * lbufp + 2 * kk, C2<T>{gv[u].x, gv[u].y});
                stc(buf + f * lbufp + 2 * kk + 1, C2<T>{gv[u].z, gv[u].w});
            }
        }
    }
    for (int e0 = d.fuse_in_r || pairs ? nf * span : threadIdx.x; e0 < nf * span; e0 += kU * kFftThreads) {
        C2<T> z[kU], cp[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + u * kFftThreads;
            z[u] = C2<T>{T(0), T(0)};
            cp[u] = C2<T>{T(1), T(0)};
            if (e < nf * span) {
                const int f = udiv(e, mg_span), k = e - f * span;
                if (k < h) {
                    z[u] = *reinterpret_cast<const C2<T> *>(gridb + (uint64_t)(unsigned)f * npts + 2u * (unsigned)k);
                    if (d.blue) cp[u] = chirp[(unsigned)k];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + u * kFftThreads;
            if (e >= nf * span) continue;
            const int f = udiv(e, mg_span), k = e - f * span;
            stc(buf + f * lbufp + k, d.blue ? cmul(z[u], cp[u]) : z[u]);
        }
    }
    if (!d.fuse_in_r) __syncthreads();
    dft_passes<T, CAP>(d, ps, d.seam_r, d.fuse_in_r, d.nrad_r - d.fuse_out_r, nf, it.shape, tw);
    // 2. split: Y_m = (Z_m + conj Z_{h-m}) / 2 - (i/2) e^{-2 pi i m / n} (Z_m - conj Z_{h-m})
    const T scale = a.adjoint ? T(1) : T(1.0 / d.n);
    C2<T> *fourb = (C2<T> *)a.out + d.four_off + f0;  // (m, f) at fourb[m nfld + f]
    const unsigned nfld = (unsigned)a.nfld;
    const unsigned mg_nf = div_magic(nf);
    if (d.fuse_out_r) {
        const FourSide<T> fs{lbufp, nf, h, M, nfld, mg_nf, (GlobalOut<T> *)fourb, (GlobalC2<T> *)post};
        const PassDesc pd = ps[d.nrad_r - 1];
        const T s0 = T(0.5) * scale, s1 = a.adjoint ? scale : s0;
        radix_dispatch<kPassToFour, sizeof(T) == 8>(pd.R, [&](auto r) __attribute__((always_inline)) {
            pass_to_four<T, decltype(r)::value>(fs, pd, (GlobalC2<T> *)W, s0, s1, smax);
        });
    }
    const int nout = d.fuse_out_r ? 0 : nf * (M + 1);
    for (int e0 = threadIdx.x; e0 < nout; e0 += kU * kFftThreads) {
        C2<T> pm[kU], cm[kU], ch[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + u * kFftThreads;
            const int m = e < nout ? udiv(e, mg_nf) : 0;
            pm[u] = post[(unsigned)m];
            cm[u] = C2<T>{T(1), T(0)};
            ch[u] = C2<T>{T(1), T(0)};
            if (d.blue) {
                // the chirp at h - m is the chirp at m times (-1)^h (m > 0)
                cm[u] = chirp[(unsigned)m];
                ch[u] = (m > 0 && (h & 1)) ? C2<T>{-cm[u].x, -cm[u].y} : cm[u];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = e0 + u * kFftThreads;
            if (e >= nout) continue;
            const int m = udiv(e, mg_nf), f = e - m * nf;
            const LdsC2<T> *sl = buf + f * lbufp;
            const C2<T> xm = ldc(sl + m), xc = ldc(sl + (m == 0 ? 0 : h - m));
            const C2<T> zm = d.blue ? cmul(cm[u], cconj(xm)) : xm;
            const C2<T> zc = cconj(d.blue ? cmul(ch[u], cconj(xc)) : xc);
            C2<T> A = cadd(zm, zc), B = csub(zm, zc);
            C2<T> t = cmul(pm[u], B);
            C2<T> y = {T(0.5) * (A.x + t.y), T(0.5) * (A.y - t.x)};
            T fac = (a.adjoint && m > 0) ? T(2) : T(1);
            y = {y.x * scale * fac, m == 0 ? T(0) : y.y * scale * fac};
            put_four<T>((GlobalOut<T> *)fourb, nfld, m, f, y, smax);
        }
    }
    if (a.fmax) {
        __syncthreads();
        for (int f = threadIdx.x; f < nf; f += kFftThreads) atomicMax(a.fmax + f0 + f, smax[f]);
    }
}

template <typename T>
bool check_fft(const Plan &p, int cap)
{
#define SHTX_FFT_FAIL                                                                    \
    do {                                                                                 \
        if (std::getenv("SHTX_DEBUG")) std::fprintf(stderr, "shtx: FFT check line %d\n", __LINE__); \
        return false;                                                                    \
    } while (0)
    if (p.fft_items.empty() || p.fft_items.size() % kXcds) SHTX_FFT_FAIL;
    size_t celem = 2 * sizeof(T);
    for (const RingDesc &d : p.rings) {
        if (d.lbuf > cap || d.L > d.lbuf || d.h + 1 > d.lbuf || d.M >= d.h) SHTX_FFT_FAIL;
        if (d.lbufp < d.lbuf) SHTX_FFT_FAIL;
        if (d.tw_off < 0 || d.tw_off + d.L > p.twid_elems) SHTX_FFT_FAIL;
        if (d.post_off < 0 || d.post_off + d.h + 1 > p.twid_elems) SHTX_FFT_FAIL;
        if (d.blue && (d.chirp_off < 0 || d.chirp_off + d.h > p.twid_elems || d.bhat_off < 0 ||
                       d.bhat_off + d.L > p.twid_elems))
            SHTX_FFT_FAIL;
        if (d.grid_off + d.n > p.npts || d.four_off + (int64_t)(d.M + 1) * p.nfld > p.nfour * p.nfld)
            SHTX_FFT_FAIL;
        // the kernels index a field's grid row and a ring's Fourier rows with
        // 32-bit unsigned element offsets
        if (p.npts >= (int64_t(1) << 32) || (int64_t)(d.M + 1) * p.nfld >= (int64_t(1) << 32)) SHTX_FFT_FAIL;
        if (d.conv && (d.conv_p < 3 || d.h % d.conv_p || d.conv_tw_off < 0 || d.conv_perm_off < 0 || d.bhat_off < 0 ||
                       std::max({d.conv_tw_off, d.conv_perm_off, d.bhat_off}) + d.conv_p - 1 > p.twid_elems))
            SHTX_FFT_FAIL;
        // both directions' pass lists: every pass of a kind with a butterfly for
        // its radix, and its descriptor exactly that pass
        int extra = 0;
        for (int dir = 0; dir < 2; ++dir) {
            const int off = dir ? d.pass_off_r : d.pass_off, nrad = dir ? d.nrad_r : d.nrad;
            const int fin = dir ? d.fuse_in_r : d.fuse_in, fout = dir ? d.fuse_out_r : d.fuse_out;
            const int seam = dir ? d.seam_r : d.seam;
            // Bluestein's seam stands between passes of both its FFTs
            if (d.blue ? seam < 1 || seam > nrad - 2 : !d.conv && seam != -1) SHTX_FFT_FAIL;
            // so does a prime pass's by convolution, whose passes come first
            if (d.conv && (d.blue || fin || d.conv > nrad || seam < 1 || seam > d.conv - 2)) SHTX_FFT_FAIL;
            if (off < 0 || nrad < 1 || off + nrad > (int)p.passes.size()) SHTX_FFT_FAIL;
            // fused passes: one pass cannot be both; Bluestein's Fourier side
            // goes through LDS
            if ((fin | fout) & ~1 || fin + fout > nrad || (d.blue && (dir ? fout : fin))) SHTX_FFT_FAIL;
            int prod = 1;
            for (int s = 0; s < nrad; ++s) {
                const PassDesc &pd = p.passes[off + s];
                const int R = pd.R;
                const bool first = s == 0 && fin, last = s == nrad - 1 && fout;
                if (s < d.conv) {
                    // transforms of length p - 1, h / p of them a field
                    const int P = d.conv_p - 1;
                    const int kind = s == 0            ? kPassGather
                                     : s == seam       ? kPassSubSeam
                                     : s == d.conv - 1 ? kPassScatter
                                                       : kPassSub;
                    if (!fft_radix_ok(kind, sizeof(T) == 8, R) || P % R || last) SHTX_FFT_FAIL;
                    if (d.fb * (d.h / d.conv_p) > kFftThreads) SHTX_FFT_FAIL;  // one extra entry a thread
                    if ((int64_t)d.fb * (d.h / d.conv_p) * (P / R) > (int64_t)fft_rounds(cap, R) * kFftThreads)
                        SHTX_FFT_FAIL;
                    if (pd.Ns != prod || pd.nbf * R != P || pd.tstep * prod * R != P) SHTX_FFT_FAIL;
                    if (pd.mg_nbf != div_magic(pd.nbf) || pd.mg_ns != div_magic(pd.Ns)) SHTX_FFT_FAIL;
                    const int cmax = R == 23 ? 17 : R == 9 ? 3 : R >= 10 ? 4 : 1;
                    if (prod > 1 && (int64_t)cmax * (prod - 1) * pd.tstep >= P) SHTX_FFT_FAIL;
                    prod *= R;
                    if ((s == seam || s == d.conv - 1) && prod != P) SHTX_FFT_FAIL;
                    if (s == seam) prod = R;
                    if (s == d.conv - 1) prod = d.conv_p;
                    continue;
                }
                const int kind = d.blue && s == seam ? kPassSeam
                                 : first   ? (dir ? kPassFromGrid : kPassFromFour)
                                 : last    ? (dir ? kPassToFour : kPassToGrid)
                                           : kPassLds;
                if (R < 2 || d.L % R) SHTX_FFT_FAIL;
                if (gp_radix(R, sizeof(T) == 8)) {
                    // a general prime pass: the first pass only, an odd prime up to
                    // kGpMaxPrime, whose output units fit one tile per wave
                    if (s != 0 || first || last || R > kGpMaxPrime || R % 2 == 0 || d.blue) SHTX_FFT_FAIL;
                    for (int q = 3; q * q <= R; q += 2)
                        if (R % q == 0) SHTX_FFT_FAIL;
                    if (!gp_best_shape(R, d.fb * pd.nbf)) SHTX_FFT_FAIL;
                    extra = R;
                } else {
                    if (!fft_radix_ok(kind, sizeof(T) == 8, R)) SHTX_FFT_FAIL;
                    if (d.blue && ((last && !blue_last_radix(R, sizeof(T) == 8)) ||
                                   (first && !blue_first_radix(R, sizeof(T) == 8))))
                        SHTX_FFT_FAIL;
                    // every butterfly of a block's fields is covered by the pass's rounds
                    if ((int64_t)d.fb * (d.L / R) > (int64_t)fft_rounds(cap, R) * kFftThreads) SHTX_FFT_FAIL;
                }
                if (pd.Ns != prod || pd.nbf * R != d.L || pd.tstep * prod * R != d.L) SHTX_FFT_FAIL;
                if (pd.mg_nbf != div_magic(pd.nbf) || pd.mg_ns != div_magic(pd.Ns)) SHTX_FFT_FAIL;
                // twiddle reads W[c k tstep], k < Ns: c = 1, and 3 for radix 9, 4 for
                // 10 to 20, 17 for the streamed radix 23
                const int cmax = R == 23 ? 17 : R == 9 ? 3 : R >= 10 ? 4 : 1;
                if (prod > 1 && (int64_t)cmax * (prod - 1) * pd.tstep >= d.L) SHTX_FFT_FAIL;
                prod *= R;
                if (d.blue && s == seam) {
                    // ends the first FFT and begins the second
                    if (prod != d.L) SHTX_FFT_FAIL;
                    prod = R;
                }
            }
            if (prod != d.L) SHTX_FFT_FAIL;
        }
        if ((size_t)(d.fb * d.lbufp + extra) * celem > (size_t)p.fft_lds_bytes)
            SHTX_FFT_FAIL;
    }
    if (p.prec == SHTX_FP16X3) {
        // the r2c kernel's per-field maxima sit after the block's LDS
        for (const RingDesc &d : p.rings)
            if (d.fb > kFmaxFields) SHTX_FFT_FAIL;
        if (p.fft_lds_bytes + 4 * kFmaxFields > 160 * 1024) SHTX_FFT_FAIL;
    }
    for (const FftItem &it : p.fft_items) {
        if (it.ring < 0) continue;
        if (it.ring >= p.nlat || it.f0 < 0 || it.nf < 1 || it.f0 + it.nf > p.nfld) SHTX_FFT_FAIL;
        const RingDesc &d = p.rings[it.ring];
        if (it.nf > d.fb) SHTX_FFT_FAIL;
        // a prime pass's tile shape has to cover the item's units
        const PassDesc &pd = p.passes[d.pass_off];
        if (!d.conv && gp_radix(pd.R, sizeof(T) == 8) && !gp_shape_ok(it.shape, pd.R, it.nf * pd.nbf))
            SHTX_FFT_FAIL;
    }
    return true;
#undef SHTX_FFT_FAIL
}

__global__ void k_zero_u32(unsigned *x, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0u;
}

// LDS words the r2c kernel adds for the per-field maxima: the largest
// fields-per-block of the plan.
int fmax_lds_bytes(const Plan &p)
{
    int fb = 0;
    for (const RingDesc &d : p.rings) fb = std::max(fb, d.fb);
    return 4 * fb;
}

template <typename T, int CAP, bool C2R>
hipError_t launch_fft(const Plan &p, const void *in, void *out, bool adjoint, unsigned *fmax, hipStream_t s)
{
    // the rings, passes and work list were checked against the kernels'
    // limits (check_fft) when the plan's blocking was built
    if (!p.shapes_ok || p.fft_items.empty()) return hipErrorInvalidValue;
    FftArgs a{p.d_rings, p.d_fft_items, p.d_passes, p.d_twid, in, out, p.nfld, adjoint ? 1 : 0, p.npts,
              nullptr, p.fft_lds_bytes};
    int lds = p.fft_lds_bytes;
    if (!C2R && p.prec == SHTX_FP16X3) {
        // per-field maxima of the Fourier workspace for the split-half GEMM:
        // cleared here (a kernel, not a memset, so that graph replays clear it)
        if (!fmax) return hipErrorInvalidValue;
        k_zero_u32<<<(p.nfld + 255) / 256, 256, 0, s>>>(fmax, p.nfld);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        a.fmax = fmax;
        lds += fmax_lds_bytes(p);
    }
    auto kern = C2R ? k_fft_c2r<T, CAP> : k_fft_r2c<T, CAP>;
    kern<<<(int)p.fft_items.size(), kFftThreads, lds, s>>>(a);
    return hipGetLastError();
}

// Dynamic LDS above 64 KiB must be allowed per kernel; allowing the whole
// workgroup LDS once (a limit, not a reservation: occupancy follows the
// LDS each launch asks for) keeps every plan's launches valid without
// per-launch attribute calls.
template <typename T, int CAP>
hipError_t fft_allow_lds()
{
    constexpr int kMaxLds = 160 * 1024;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_fft_c2r<T, CAP>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_fft_r2c<T, CAP>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    return e;
}

}  // namespace

hipError_t fft_prepare(const Plan &p)
{
    if (p.fft_lds_bytes > 160 * 1024) return hipErrorInvalidValue;
    return p.prec == SHTX_FP64 ? fft_allow_lds<double, kFftCapF64>() : fft_allow_lds<float, kFftCapF32>();
}

bool fft_shapes_ok(const Plan &p)
{
    bool ok = p.prec == SHTX_FP64 ? check_fft<double>(p, kFftCapF64) : check_fft<float>(p, kFftCapF32);
    if (!ok && std::getenv("SHTX_DEBUG")) std::fprintf(stderr, "shtx: ring-FFT launch shape check failed\n");
    return ok;
}

hipError_t launch_fft_c2r(const Plan &p, const void *four, void *grid, bool adjoint, hipStream_t s)
{
    if (p.prec == SHTX_FP64) return launch_fft<double, kFftCapF64, true>(p, four, grid, adjoint, nullptr, s);
    return launch_fft<float, kFftCapF32, true>(p, four, grid, adjoint, nullptr, s);
}

hipError_t launch_fft_r2c(const Plan &p, const void *grid, void *four, bool adjoint, unsigned *fmax, hipStream_t s)
{
    if (p.prec == SHTX_FP64) return launch_fft<double, kFftCapF64, false>(p, grid, four, adjoint, nullptr, s);
    return launch_fft<float, kFftCapF32, false>(p, grid, four, adjoint, fmax, s);
}

}  // namespace shtx
