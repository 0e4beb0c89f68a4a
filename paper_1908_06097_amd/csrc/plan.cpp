// Plan construction for libshtx: ring geometry, Legendre table layout, GEMM
// and ring-FFT work lists, FFT twiddle tables, device allocations, and the
// device-side generation of Gauss nodes and P̄_n^m tables.
//
// The paper (Section 3.1.1) keeps the transform's data resident on the GPU
// across time steps; here everything a transform needs (tables, twiddles,
// work lists, the Fourier workspace) is allocated once per plan so that the
// transform calls themselves never allocate.
#include <array>
#include <chrono>
#include <cmath>
#include <complex>
#include <cstring>
#include <map>

#include "shtx_internal.h"

namespace shtx {

namespace {

int ring_cutoff(int trunc, int nlon)
{
    int m = (nlon - 1) / 2;
    return m < trunc ? m : trunc;
}

int64_t round_up(int64_t x, int64_t q) { return (x + q - 1) / q * q; }

// Radices the ring-FFT kernel implements directly (primes; 4, 8, 9 and 16
// are formed from the factors of 2 and 3).  FP64 plans stop at 17.
const int kPrimeRadices[] = {2, 3, 5, 7, 11, 13, 17, 19, 23};

// Factor n over the direct prime radices up to maxp; returns the unfactored
// remainder.
int smooth_factor(int n, std::vector<int> &f, int maxp = 23)
{
    f.clear();
    for (int p : kPrimeRadices)
        while (p <= maxp && n % p == 0) {
            f.push_back(p);
            n /= p;
        }
    return n;
}

bool is_prime(int n)
{
    if (n < 2) return false;
    for (int q = 2; q * q <= n; ++q)
        if (n % q == 0) return false;
    return true;
}

// Cost model of a ring FFT's passes, in vector instructions per complex value
// (counted from the butterflies' additions and multiply-adds), by which the
// plan picks a ring length's radices.

// Radix-R butterfly in registers.
double butterfly_cost(int R)
{
    switch (R) {
    case 2: return 2;
    case 4: return 4;
    case 8: return 6.75;
    case 9: return 11.2;
    case 16: return 10.2;
    case 6: case 10: case 14: return 2 + butterfly_cost(R / 2);
    case 18: return 2 + butterfly_cost(9);
    case 12: case 20: return 4 + butterfly_cost(R / 4);
    case 15: return butterfly_cost(3) + butterfly_cost(5);
    }
    const double H = (R - 1) / 2;  // odd primes, inputs paired
    return (4 * H * H + 10 * H) / R;
}

// How often the lanes of a pass's LDS writes meet in a bank pair: the most of
// 64 consecutive butterflies that fall on one of the 32 pairs, over the two
// that have to.
double write_conflicts(int R, int Ns, int nbf)
{
    int load[32] = {0}, top = 0, n = std::min(64, nbf);
    for (int j = 0, a = 0, r = 0; j < n; ++j) {  // a = (j / Ns) Ns R + j % Ns
        top = std::max(top, ++load[a % 32]);
        ++a;
        if (++r == Ns) {
            r = 0;
            a += Ns * (R - 1);
        }
    }
    return std::max(1.0, top / 2.0);
}

// One pass: butterfly and twiddles, per-butterfly index work, and for a pass
// in LDS its write, its barriers and the conflicts of its writes; a pass that
// writes to memory needs none of the latter.
double pass_cost(int R, int Ns, int nbf, bool to_lds)
{
    double c = butterfly_cost(R) + 30.0 / R + 4;
    if (Ns > 1) c += 8.0 * (R - 1) / R;
    if (to_lds) c += 8 + 3 * (write_conflicts(R, Ns, nbf) - 1);
    return c;
}

// The passes of a ring FFT of length L in one direction.
struct PassPlan {
    std::vector<int> rad;
    int fuse_in = 0, fuse_out = 0, seam = -1;
    double cost = 1e300;  // vector instructions per value, idle lanes counted
};

constexpr double kUnfused = 12;  // a separate loop for the reads or writes

// Lanes without a butterfly in a pass's rounds hide less latency: a quarter of
// their share counts (half picked more passes of smaller radices, and rings of 4076
// points, 411 fields, took 9.0 instead of 8.3 ps per point).
double idle_factor(int butterflies)
{
    const int lanes = (butterflies + kFftThreads - 1) / kFftThreads * kFftThreads;
    return 0.75 + 0.25 * lanes / butterflies;
}

// The cheapest passes that bring a length-L FFT from stride Ns0 to stride Ns1
// (the product of the radices so far): every ordered factorisation with a
// butterfly for each pass's kind.  kin, kout: kinds that the first and the last
// of them may take instead of LDS (kPassLds: none).  fields: per block.  No
// passes if none cost less than `limit`.
PassPlan order_passes(int L, int Ns0, int Ns1, int kin, int kout, int fields, bool dbl, bool blue, double limit = 1e300)
{
    PassPlan best;
    best.cost = limit;
    std::vector<int> cur;
    auto go = [&](auto &&self, int Ns, double cost, int fuse_in) -> void {
        const int left = Ns1 / Ns;
        // no pass costs less than 7 log2(R), 8 of them its writes and 8 its twiddles
        if (cost + std::max(10.0, 7.0 * std::log2(left) - (Ns == 1 ? 16 : 8)) >= best.cost) return;
        for (int R = kTopRadix; R >= 2; --R) {
            if (left % R) continue;
            const int nbf = L / R;
            const bool last = left == R;
            cur.push_back(R);
            auto step = [&](int kind, bool fin, bool fout) {
                // one field's butterflies have to fit the pass's rounds
                if (!fft_radix_ok(kind, dbl, R) ||
                    nbf > fft_rounds(dbl ? kFftCapF64 : kFftCapF32, R) * kFftThreads)
                    return;
                if (blue && ((fin && !blue_first_radix(R, dbl)) || (fout && !blue_last_radix(R, dbl)))) return;
                const double idle = blue ? idle_factor(nbf * fields) : 1.0;
                if (cost + idle * pass_cost(R, Ns, nbf, false) >= best.cost) return;  // before the conflicts
                double c = cost + idle * pass_cost(R, Ns, nbf, !fout);
                if (Ns == 1 && kin != kPassLds && !fin) c += kUnfused;
                if (last) {
                    if (kout != kPassLds && !fout) c += kUnfused;
                    if (c < best.cost) {
                        best.cost = c;
                        best.rad = cur;
                        best.fuse_in = fin || fuse_in;
                        best.fuse_out = fout;
                    }
                } else if ((int)cur.size() < kMaxRadices - 1) {
                    self(self, Ns * R, c, fin || fuse_in);
                }
            };
            if (Ns == 1 && kin != kPassLds && (!last || blue)) step(kin, true, false);
            step(kPassLds, false, false);
            if (last && kout != kPassLds) step(kout, false, true);
            cur.pop_back();
        }
    };
    if (Ns0 == Ns1)
        best.cost = 0;
    else
        go(go, Ns0, 0.0, 0);
    return best;
}

// Passes of a plain FFT of length L, after a first pass of radix `lead` (1:
// none) that ran already, in LDS.
PassPlan plan_passes(int L, int lead, bool r2c, bool dbl)
{
    PassPlan p = order_passes(L, lead, L, lead > 1 ? kPassLds : r2c ? kPassFromGrid : kPassFromFour,
                              r2c ? kPassToFour : kPassToGrid, 1, dbl, false);
    if (lead > 1) p.rad.insert(p.rad.begin(), lead);
    return p;
}

// Bluestein's passes of length L in one direction: the first FFT up to its last
// pass, the seam, and the rest of the second FFT, for the cheapest radix of
// the seam; the r2c kernel's first pass reads the grid and the c2r kernel's
// last one writes it.
PassPlan bluestein_passes(int L, bool r2c, bool dbl)
{
    PassPlan best;
    const int cap = dbl ? kFftCapF64 : kFftCapF32, fields = std::max(1, cap / L);
    for (int J = kTopRadix; J >= 2; --J) {
        if (L % J || L == J || !fft_radix_ok(kPassSeam, dbl, J) || L / J > fft_rounds(cap, J) * kFftThreads) continue;
        const double seam = idle_factor(L / J * fields) * (pass_cost(J, 2, L / J, true) + butterfly_cost(J) + 8 +
                                                           3 * (write_conflicts(J, 1, L / J) - 1));
        const PassPlan a = order_passes(L, 1, L / J, r2c ? kPassFromGrid : kPassLds, kPassLds, fields, dbl, true,
                                        best.cost - seam - 10);
        if (a.rad.empty()) continue;
        const PassPlan b = order_passes(L, J, L, kPassLds, r2c ? kPassLds : kPassToGrid, fields, dbl, true,
                                        best.cost - seam - a.cost);
        if (b.rad.empty()) continue;
        best = a;
        best.seam = (int)a.rad.size();
        best.rad.push_back(J);
        best.rad.insert(best.rad.end(), b.rad.begin(), b.rad.end());
        best.fuse_out = b.fuse_out;
        best.cost = a.cost + b.cost + seam;
    }
    return best;
}

// Passes of a prime pass by convolution: two FFTs of length P = p - 1 around a
// seam, their first pass a gather and their last a scatter; no passes if P has
// no such factors.  per: transforms a field, fields: a block.
PassPlan conv_passes(int p, int per, int fields, bool dbl)
{
    constexpr double kPermute = 6;  // table reads and LDS conflicts of a permuted side
    const int P = p - 1, cap = dbl ? kFftCapF64 : kFftCapF32;
    PassPlan best;
    auto fits = [&](int kind, int R) {
        return fft_radix_ok(kind, dbl, R) && fields * per * (P / R) <= fft_rounds(cap, R) * kFftThreads;
    };
    auto cost = [&](int R, int Ns) { return idle_factor(fields * per * (P / R)) * pass_cost(R, Ns, P / R, true); };
    for (int J = kTopRadix; J >= 2; --J) {
        if (P % J || !fits(kPassSubSeam, J)) continue;
        const double seam = cost(J, 2) + idle_factor(fields * per * (P / J)) * (butterfly_cost(J) + 8);
        // the other factor in one to three passes, those of the second FFT
        // after a product of J
        PassPlan half[2];
        for (int out = 0; out < 2; ++out) {
            std::vector<int> cur;
            auto go = [&](auto &&self, int left, int Ns, double c) -> void {
                for (int R = kTopRadix; R >= 2; --R) {
                    if (left % R) continue;
                    const int kind = out ? (left == R ? kPassScatter : kPassSub) : (cur.empty() ? kPassGather : kPassSub);
                    if (!fits(kind, R)) continue;
                    const double cr = c + cost(R, Ns);
                    if (cr >= half[out].cost) continue;
                    cur.push_back(R);
                    if (left == R) {
                        half[out].cost = cr;
                        half[out].rad = cur;
                    } else if (cur.size() < 3) {
                        self(self, left / R, Ns * R, cr);
                    }
                    cur.pop_back();
                }
            };
            go(go, P / J, out ? J : 1, kPermute);
        }
        if (half[0].rad.empty() || half[1].rad.empty() || half[0].cost + half[1].cost + seam >= best.cost) continue;
        best.cost = half[0].cost + half[1].cost + seam;
        best.rad = half[0].rad;
        best.seam = (int)best.rad.size();
        best.rad.push_back(J);
        best.rad.insert(best.rad.end(), half[1].rad.begin(), half[1].rad.end());
    }
    return best;
}

int primitive_root(int p)
{
    for (int g = 2;; ++g) {
        int k = 1;
        for (int64_t x = g; x != 1; x = x * g % p) ++k;
        if (k == p - 1) return g;
    }
}

// Both directions' passes of a Bluestein length, made once per length.
struct BluePlan {
    PassPlan pass[2];
    double cost = 1e300;
};

// The cheapest Bluestein length from lo to cap (factors up to 7) and its cost
// per field and value, with its passes in `plans`.
std::pair<double, int> bluestein_length(int lo, int cap, bool dbl, std::map<int, BluePlan> &plans)
{
    std::pair<double, int> best = {1e300, 0};
    for (int L = lo; L <= cap && L <= lo + lo / 8 + 32; ++L) {
        int y = L;
        for (int q : {2, 3, 5, 7})
            while (y % q == 0) y /= q;
        if (y != 1) continue;
        auto it = plans.find(L);
        if (it == plans.end()) {
            BluePlan b;
            for (int dir = 0; dir < 2; ++dir) b.pass[dir] = bluestein_passes(L, dir == 1, dbl);
            b.cost = 0.5 * (b.pass[0].cost + b.pass[1].cost);
            it = plans.emplace(L, b).first;
        }
        if (it->second.cost * L < best.first * best.second || !best.second) best = {it->second.cost, L};
    }
    return best;
}

template <class T>
hipError_t upload(T **dst, const std::vector<T> &src)
{
    if (src.empty()) {
        *dst = nullptr;
        return hipSuccess;
    }
    hipError_t e = hipMalloc(dst, sizeof(T) * src.size());
    if (e != hipSuccess) return e;
    return hipMemcpy(*dst, src.data(), sizeof(T) * src.size(), hipMemcpyHostToDevice);
}

}  // namespace

// Default tiles.  128 x 128 but where rows or columns would mostly be padding;
// measured on octahedral grids, microseconds at 128 x 128 / 64 x 128 / 128 x 64:
//   few rows a wavenumber: FP32 inverse T213 37 fields 28 / 22 / 23, T639 40
//   fields 225 / 228; BF16x3 inverse T213 20 / 17, T639 411 fields 1120 / 1270;
//   direct FP32 T255 411 fields 190 / 177, T639 1684 / 1824, BF16x3 T399 137
//   fields 188 / 174, T639 411 fields 1173 / 1316;
//   columns: FP32 inverse T639 137 fields (274 columns in 384 or 320) 599 / 629
//   / 544, T1279 4096 / 4553 / 3856, but 411 fields (822 in 896 or 832) 10043 /
//   11427 / 10561.
void gemm_tiles(int prec, int trunc, int nfld, int *inv_bm, int *inv_bn, int *dir_bm, int *dir_bn)
{
    if (prec == SHTX_FP64) {
        *inv_bm = 64; *inv_bn = 64; *dir_bm = 64; *dir_bn = 64;
        return;
    }
    const int64_t by64 = round_up(2 * nfld, 64), by128 = round_up(2 * nfld, 128);
    *inv_bm = trunc < 240 ? 64 : 128;
    *inv_bn = prec == SHTX_FP32 && trunc >= 240 && 9 * by64 < 8 * by128 ? 64 : 128;
    *dir_bm = trunc < 512 ? 64 : 128;
    *dir_bn = 128;
}

// Long-double mixed-radix DFT (forward), used once per ring length at plan time
// for the Bluestein filter spectrum.  tw: the N-th roots of unity, n | N.
using cld = std::complex<long double>;
static cld mul(const cld &a, const cld &b)
{
    return {a.real() * b.real() - a.imag() * b.imag(), a.real() * b.imag() + a.imag() * b.real()};
}
static void dft_ld(cld *x, int n, const std::vector<cld> &tw, int N)
{
    if (n == 1) return;
    int p = 2;
    for (int q : {2, 3, 5, 7, 11, 13, 17, 19, 23})
        if (n % q == 0) {
            p = q;
            break;
        }
    const int m = n / p, step = N / n;  // tw[t step] = exp(-2 pi i t / n)
    // decimation in time: sub-sequence r holds x[k p + r]
    std::vector<cld> sub((size_t)n);
    for (int r = 0; r < p; ++r)
        for (int k = 0; k < m; ++k) sub[(size_t)r * m + k] = x[(size_t)k * p + r];
    for (int r = 0; r < p; ++r) dft_ld(sub.data() + (size_t)r * m, m, tw, N);
    cld b[23];
    for (int k = 0; k < m; ++k) {
        b[0] = sub[k];
        for (int r = 1; r < p; ++r) b[r] = mul(sub[(size_t)r * m + k], tw[(size_t)r * k * step]);
        if (p == 2) {
            x[k] = b[0] + b[1];
            x[k + m] = b[0] - b[1];
            continue;
        }
        cld sum = b[0];  // p odd: outputs q and p - q from the pairs r and p - r
        for (int r = 1; r < p; ++r) sum += b[r];
        x[k] = sum;
        for (int q = 1; q <= p / 2; ++q) {
            cld u = b[0], v = 0;
            for (int r = 1; r <= p / 2; ++r) {
                const cld w = tw[(size_t)(r * q % p) * (N / p)];
                u += w.real() * (b[r] + b[p - r]);
                v += w.imag() * (b[r] - b[p - r]);
            }
            x[(size_t)q * m + k] = {u.real() - v.imag(), u.imag() + v.real()};
            x[(size_t)(p - q) * m + k] = {u.real() + v.imag(), u.imag() - v.real()};
        }
    }
}

// Bluestein's filter: DFT_L(b) / L in long double, b the conjugate chirp of
// half-length h wrapped to length L, from the plan's twiddles of L and chirp
// (interleaved).
static void bluestein_filter(int h, int L, const long double *twid, const long double *chirp,
                             std::vector<long double> &re, std::vector<long double> &im)
{
    std::vector<cld> b((size_t)L, 0), tw((size_t)L);
    for (int k = 0; k < L; ++k) tw[k] = {twid[2 * k], twid[2 * k + 1]};
    for (int j = 0; j < h; ++j) {
        b[j] = {chirp[2 * j], -chirp[2 * j + 1]};
        if (j > 0) b[L - j] = b[j];
    }
    dft_ld(b.data(), L, tw, L);
    re.resize(L);
    im.resize(L);
    for (int k = 0; k < L; ++k) {
        re[k] = b[k].real() / L;
        im[k] = b[k].imag() / L;
    }
}

void free_plan(Plan &p)
{
    void *ptrs[] = {p.d_mu, p.d_w, p.d_diag, p.d_tab_inv, p.d_tab_dir, p.d_mmax, p.d_mb, p.d_inv_items, p.d_dir_items,
                    p.d_rings, p.d_ring_four_off, p.d_ring_pair, p.d_ring_q, p.d_fft_items, p.d_passes,
                    p.d_twid, p.d_four, p.d_fmax, p.d_diag_e, p.d_uvspec};
    for (void *q : ptrs)
        if (q) (void)hipFree(q);
    for (auto &g : p.graphs)
        if (g.exec) (void)hipGraphExecDestroy(g.exec);
    for (auto e : p.ev_start) (void)hipEventDestroy(e);
    for (auto e : p.ev_stop) (void)hipEventDestroy(e);
    if (p.done) (void)hipEventDestroy(p.done);
    p = Plan();
}

#define PLAN_TRY(expr)                                   \
    do {                                                 \
        hipError_t e_ = (expr);                          \
        if (e_ != hipSuccess) {                          \
            (void)hipGetLastError();                     \
            return e_ == hipErrorOutOfMemory ? SHTX_ENOMEM : SHTX_EHIP; \
        }                                                \
    } while (0)

namespace {

// How a ring's FFT runs: without large primes, with a general prime pass, with a
// prime pass by convolution, by Bluestein.
enum RingKind { kRingPlain, kRingPrime, kRingConv, kRingBlue };

// Time of one block of nf fields of a ring of half-length h, in nanoseconds with
// the CUs full of such blocks: so much for the block (its descriptors, first
// loads, last stores), for each pass (barriers and the loads it begins with;
// `passes` without a general prime pass), for each value, and for the work of
// the kind's own: a prime pass's cycles (16 p for each unit of a wave),
// instructions per value of a convolution's or Bluestein's passes.  Fitted to
// 10 494 timings on MI355X (random lengths of 20 to 16 382 points, 1 to 411
// fields, every kind that a length can take; 6 to 11 % RMS).  A block of few
// values is mostly its passes, of which a convolution and Bluestein have more:
// by throughput alone, as 411 fields have it, some rings of few fields ran up
// to half as long again (us, general prime pass | convolution | Bluestein, both
// directions, 512 rings; FP64 244 points, 2 fields, 24.4 | 36.8 | 38.6; FP32 122
// points, 3 fields, 17.6 | 24.1 | 21.9; but FP32 2416 points, 411 fields, 4.2 |
// 3.1 | - ps per point).  With it the choice costs 0.2 % against the fastest of
// the three on average over the timed rings, 2.5 % before.
double block_time(bool dbl, RingKind kind, int h, double passes, int nf, double work)
{
    static const double t[2][4][4] = {{{2800, 280, 1.23, 0}, {3000, 830, 1.24, 1.0}, {3700, 560, 1.37, 0.0059},
                                       {6000, 290, 1.44, 0.0055}},
                                      {{3200, 280, 1.23, 0}, {3200, 710, 1.46, 0.91}, {3400, 590, 1.27, 0.0073},
                                       {4600, 600, 1.97, 0.0039}}};
    const double *c = t[dbl][kind];
    return c[0] + c[1] * passes + c[2] * h * nf + c[3] * work;
}

// Of F fields, fb a block (the last block takes what is left).
template <class Fn>
double fields_time(int F, int fb, Fn block)
{
    return F / fb * block(fb) + (F % fb ? block(F % fb) : 0.0);
}

double prime_block_time(bool dbl, int p, int h, double passes, int nf)
{
    return block_time(dbl, kRingPrime, h, passes, nf, 16.0 * p * gp_cost(gp_best_shape(p, nf * (h / p))));
}

// By what a ring's ways of running are compared: the time of nlat such rings on
// the chip's block slots (two a CU, FP64 one), one block's at least.
template <class Fn>
double ring_time(bool dbl, int nlat, int F, int fb, Fn block)
{
    return std::max(block(std::min(F, fb)), fields_time(F, fb, block) * nlat / (dbl ? 256 : 512));
}

// Fields per block (at most fb) of a ring with a general prime pass, among the
// counts whose units fit one tile per wave: the least time.  Small plans, with
// slots to spare, take fewer than the most that fit (c2r, against the least time
// of the blocks' sum: T75, 45 fields on a full grid 16.2 -> 11.0 us, T117, 59 fields on
// O118 20.6 -> 18.7).  0 if not even one field's fit.
int prime_fields(bool dbl, int nlat, int p, int h, double passes, int F, int fb)
{
    int best = 0;
    double least = 0;
    for (int nf = 1; nf <= fb && gp_best_shape(p, nf * (h / p)); ++nf) {
        const double t = ring_time(dbl, nlat, F, nf, [&](int k) { return prime_block_time(dbl, p, h, passes, k); });
        if (!best || t < least) {
            best = nf;
            least = t;
        }
    }
    return best;
}

}  // namespace

// FFT blocking: fields per block (at most `cap` complex values of LDS per
// block), the XCD-segmented work list and the dynamic LDS size.
int fft_blocking(Plan &p, int cap)
{
    const int F = p.nfld, maxcap = p.prec == SHTX_FP64 ? kFftCapF64 : kFftCapF32;
    const size_t celem = p.prec == SHTX_FP64 ? 16 : 8;
    if (cap < 1 || cap > maxcap) return SHTX_EINVAL;
    int lds_elems = 0;
    std::vector<std::vector<FftItem>> fgroups;
    std::vector<double> fcost;
    std::map<std::pair<int, int>, int> prime_lim;  // by ring length and fields
    for (int j = 0; j < p.nlat; ++j) {
        RingDesc &d = p.rings[j];
        if (d.lbuf > maxcap) return SHTX_EUNSUPPORTED;
        d.fb = std::max(1, std::min(F, cap / d.lbuf));
        // a general prime pass takes one tile of output units per wave, a
        // pass in LDS its rounds of kFftThreads butterflies
        int extra = 0, gp = 0, gp_nbf = 0;
        const bool dbl = p.prec == SHTX_FP64;
        const double passes = 0.5 * (d.nrad + d.nrad_r);
        for (int dir = 0; dir < 2; ++dir) {
            const int nrad = dir ? d.nrad_r : d.nrad;
            for (int s = 0; s < nrad; ++s) {
                const PassDesc &q = p.passes[(dir ? d.pass_off_r : d.pass_off) + s];
                const int R = q.R;
                int lim;
                if (s < d.conv) {
                    lim = std::min(fft_rounds(maxcap, R) * kFftThreads / q.nbf, kFftThreads) / (d.h / d.conv_p);
                } else if (gp_radix(R, dbl)) {
                    int &nf = prime_lim[{d.n, d.fb}];
                    if (!nf) nf = prime_fields(dbl, p.nlat, R, d.h, passes - 1, F, d.fb);
                    lim = nf;
                    extra = gp = R;
                    gp_nbf = q.nbf;
                } else {
                    lim = fft_rounds(maxcap, R) * kFftThreads / q.nbf;
                }
                if (lim < 1) return SHTX_EUNSUPPORTED;
                d.fb = std::min(d.fb, lim);
            }
        }
        lds_elems = std::max(lds_elems, d.fb * d.lbufp + extra);
        std::vector<FftItem> g;
        for (int f0 = 0; f0 < F; f0 += d.fb) {
            const int nf = std::min(d.fb, F - f0);
            g.push_back(FftItem{j, f0, nf, gp ? gp_best_shape(gp, nf * gp_nbf) : 0});
        }
        fgroups.push_back(g);
        fcost.push_back(fields_time(F, d.fb, [&](int nf) {
            return gp       ? prime_block_time(dbl, gp, d.h, passes - 1, nf)
                   : d.conv ? block_time(dbl, kRingConv, d.h, passes, nf, (double)nf * d.h * d.blue_cost)
                   : d.blue ? block_time(dbl, kRingBlue, d.h, passes, nf, (double)nf * d.L * d.blue_cost)
                            : block_time(dbl, kRingPlain, d.h, passes, nf, 0.0);
        }));
    }
    p.fft_lds_bytes = lds_elems * (int)celem;
    p.fft_lds_max = lds_elems;
    p.fft_cap = cap;
    if (p.fft_lds_bytes > 160 * 1024) return SHTX_EUNSUPPORTED;
    p.fft_items = layout_by_xcd(fgroups, fcost, FftItem{-1, 0, 0, 0});
    return SHTX_OK;
}

// GEMM work lists for the plan's current tile shapes: every (m, row tile,
// column tile), one XCD segment per group of tiles sharing an m.
int gemm_work_lists(Plan &p)
{
    if (!gemm_tile_supported(p.prec, p.inv_bm, p.inv_bn) || !gemm_tile_supported(p.prec, p.dir_bm, p.dir_bn))
        return SHTX_EUNSUPPORTED;
    if (kTablePad % p.inv_bm || kTablePad % p.dir_bm) return SHTX_EUNSUPPORTED;
    const int N = p.trunc, ncol = 2 * p.nfld;
    const int inv_bm = p.inv_narrow ? kNarrowRows : p.inv_bm, inv_bn = p.inv_narrow ? 16 * p.inv_narrow : p.inv_bn;
    const int dir_bm = p.dir_narrow ? kNarrowRows : p.dir_bm, dir_bn = p.dir_narrow ? 16 * p.dir_narrow : p.dir_bn;
    std::vector<std::vector<GemmItem>> gi, gd;
    std::vector<double> ci, cd;
    for (int m = 0; m <= N; ++m) {
        const MBlock &b = p.mb[m];
        std::vector<GemmItem> a, c;
        const int ntc_i = (ncol + inv_bn - 1) / inv_bn, ntr_i = (b.R + inv_bm - 1) / inv_bm;
        for (int tr = 0; tr < ntr_i; ++tr)
            for (int tc = 0; tc < ntc_i; ++tc) a.push_back(GemmItem{m, tr, tc, 0});
        const int ntc_d = (ncol + dir_bn - 1) / dir_bn, ntk_d = (b.K0 + dir_bm - 1) / dir_bm;
        for (int tk = 0; tk < ntk_d; ++tk)
            for (int tc = 0; tc < ntc_d; ++tc) c.push_back(GemmItem{m, tk, tc, 0});
        // a tile's K stages, and about six more for its start and its output
        if (!a.empty()) {
            ci.push_back((double)a.size() * (b.K0 / 16.0 + 6));
            gi.push_back(a);
        }
        cd.push_back((double)c.size() * (b.R / 16.0 + 6));
        gd.push_back(c);
    }
    p.inv_items = layout_by_xcd(gi, ci, GemmItem{-1, 0, 0, 0});
    p.dir_items = layout_by_xcd(gd, cd, GemmItem{-1, 0, 0, 0});
    return SHTX_OK;
}

// Host part of plan construction: geometry, table layout, FFT length plans
// and twiddle tables (kept on the host until uploaded), GEMM and FFT work
// lists.  Touches no device state, so it can be checked on any machine.
int plan_layout(Plan &p, int trunc, int grid, int nlat, int nlon_full, int nfld, int prec, unsigned flags)
{
    if (trunc < 0 || nfld < 1 || nlat < 2) return SHTX_EINVAL;
    if (grid != SHTX_GRID_FULL && grid != SHTX_GRID_OCTAHEDRAL) return SHTX_EINVAL;
    if (prec != SHTX_FP64 && prec != SHTX_FP32 && !split_form(prec)) return SHTX_EINVAL;
    if (nlat % 2) return SHTX_EUNSUPPORTED;
    if (grid == SHTX_GRID_FULL && (nlon_full < 2 || nlon_full % 2)) return nlon_full < 2 ? SHTX_EINVAL : SHTX_EUNSUPPORTED;
    if (trunc > 4095 || nlat > 16384 || nfld > (1 << 20)) return SHTX_EUNSUPPORTED;
    // wind images: truncation N + 1 >= 1 and fields U then V
    if ((flags & SHTX_FLAG_UV) && (trunc < 1 || nfld % 2)) return SHTX_EINVAL;

    p.trunc = trunc;
    p.grid = grid;
    p.nlat = nlat;
    p.nlon_full = nlon_full;
    p.nfld = nfld;
    p.prec = prec;
    p.flags = flags;
    const int N = trunc, NL = nlat / 2, F = nfld;

    // ---- ring geometry ----------------------------------------------------
    p.nlon.resize(nlat);
    p.cutoff.resize(nlat);
    for (int j = 0; j < nlat; ++j) {
        int i = j < NL ? j : nlat - 1 - j;
        p.nlon[j] = grid == SHTX_GRID_FULL ? nlon_full : 20 + 4 * i;
        p.cutoff[j] = ring_cutoff(N, p.nlon[j]);
        p.max_nlon = std::max(p.max_nlon, p.nlon[j]);
    }
    // The Legendre GEMM rows are the band of northern rings carrying m; it is
    // contiguous because the cutoff never decreases towards the equator.
    for (int j = 1; j < NL; ++j)
        if (p.cutoff[j] < p.cutoff[j - 1]) return SHTX_EUNSUPPORTED;
    p.nspec = (int64_t)(N + 1) * (N + 2) / 2;

    // ---- m blocks -----------------------------------------------------------
    p.mb.resize(N + 1);
    int64_t off = 0;
    double flops = 0.0;
    for (int m = 0; m <= N; ++m) {
        MBlock b{};
        int j0 = NL;
        for (int j = 0; j < NL; ++j)
            if (p.cutoff[j] >= m) {
                j0 = j;
                break;
            }
        b.R = NL - j0;
        b.j0 = j0;
        b.K0 = (N - m) / 2 + 1;
        b.K1 = (N - m + 1) / 2;
        b.Rp = (int)round_up(std::max(b.R, 1), kTablePad);
        b.Kp = (int)round_up(b.K0, kTablePad);
        b.e = prec == SHTX_FP32 ? kF32TableExp : 0;  // the split forms' are set with the tables
        b.off = off;
        off += 2 * (int64_t)b.Kp * b.Rp;
        p.mb[m] = b;
        flops += 4.0 * F * (double)b.R * (N - m + 1);
    }
    p.tab_elems = off;
    p.legendre_flops = flops;

    p.inv_narrow = gemm_narrow(prec, F, true);
    p.dir_narrow = gemm_narrow(prec, F, false);
    p.table_bytes = (table_entry_bytes(p, true) + table_entry_bytes(p, false)) * p.tab_elems;

    // ---- ring FFT plans and twiddle pool --------------------------------------
    const bool dbl = prec == SHTX_FP64;
    const int cap = dbl ? kFftCapF64 : kFftCapF32;
    struct LenPlan {
        int L, blue, pass_off[2];  // c2r, r2c
        PassPlan pass[2];
        int64_t tw, post, chirp, bhat;
        PassPlan conv;
        int conv_p = 0;
        int64_t conv_tw = 0, conv_perm = 0;
    };
    std::map<int, LenPlan> lens;
    std::map<int, BluePlan> blues;
    std::map<int, std::array<int64_t, 3>> convs;  // by prime: W_P, spectrum, permutations
    std::map<int, int64_t> tws;  // first root of unity by length
    std::vector<long double> pool;  // interleaved re, im
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int j = 0; j < nlat; ++j) {
        int n = p.nlon[j];
        if (lens.count(n)) continue;
        int h = n / 2;
        LenPlan lp{};
        std::vector<int> f;
        const int maxp = dbl ? 17 : 23;
        const int rem = smooth_factor(h, f, maxp);
        // A length takes Bluestein if a 2^a 3^b >= 2h - 1 with 9 | L (or 2^a 3^b
        // 5^c, for the longest TCo1999 rings) fits the LDS cap; the length and
        // passes used are the cheapest among those of factors up to 7.
        auto smallest = [](int lo, bool fives) {
            for (int x = lo;; ++x) {
                int y = x, threes = 0;
                while (y % 2 == 0) y /= 2;
                while (y % 3 == 0) y /= 3, ++threes;
                while (fives && y % 5 == 0) y /= 5;
                if (y == 1 && threes >= 2) return x;
            }
        };
        int Lb = smallest(2 * h - 1, false);
        if (Lb > cap) Lb = smallest(2 * h - 1, true);
        std::pair<double, int> bl = {1e300, 0};  // cost of a field, length
        if (rem > 1 && Lb <= cap) bl = bluestein_length(2 * h - 1, cap, dbl, blues);
        // one prime factor above the register radices runs as the first pass, as
        // a general prime pass (up to kGpMaxPrime, where one field's output units
        // fit the block's waves) or by convolution, or the whole length by
        // Bluestein: what takes the least time for the plan's fields
        const int fmost = std::max(1, std::min(F, cap / (h + 1)));
        const bool prime = rem > 1 && is_prime(rem);
        const bool can_gp = prime && rem <= kGpMaxPrime &&
                            gp_row_tiles(rem) * gp_col_tiles(h / rem) <= kGpFieldUnits && gp_best_shape(rem, h / rem);
        RingKind kind = rem == 1 ? kRingPlain : kRingBlue;
        PassPlan first[2];  // a prime pass and the others, alike for the first two ways
        if (prime && (can_gp || Lb <= cap)) {
            // passes of radix 13, 14 and 15 run one round of butterflies: with
            // them a block takes fewer fields than its LDS holds (2504 points,
            // 411 fields, 6.0 -> 4.0 ps per point), unless that splits a call's
            // few fields over two blocks (O1280, 3 fields, 108 -> 113 us)
            int conv_nf = fmost;
            lp.conv = conv_passes(rem, h / rem, conv_nf, dbl);
            if (lp.conv.rad.empty() && fmost < F && kFftThreads * 13 / h > 0) {
                conv_nf = std::min(fmost, kFftThreads * 13 / h);
                lp.conv = conv_passes(rem, h / rem, conv_nf, dbl);
            }
            conv_nf = std::min(conv_nf, std::max(1, kFftThreads / (h / rem)));
            // with `rest` passes after the prime one
            auto fastest = [&](double rest) {
                RingKind best = kRingBlue;
                double least = 1e300;
                auto take = [&](RingKind k, double t) {
                    if (t < least) {
                        best = k;
                        least = t;
                    }
                };
                if (can_gp)
                    take(kRingPrime, ring_time(dbl, nlat, F, prime_fields(dbl, nlat, rem, h, rest, F, fmost),
                                               [&](int nf) { return prime_block_time(dbl, rem, h, rest, nf); }));
                if (!lp.conv.rad.empty())
                    take(kRingConv, ring_time(dbl, nlat, F, conv_nf, [&](int nf) {
                             return block_time(dbl, kRingConv, h, rest + lp.conv.rad.size(), nf,
                                               (double)nf * h * lp.conv.cost);
                         }));
                if (Lb <= cap && bl.second) {
                    const BluePlan &b = blues[bl.second];
                    const double passes = 0.5 * (b.pass[0].rad.size() + b.pass[1].rad.size());
                    take(kRingBlue,
                         ring_time(dbl, nlat, F, std::max(1, std::min(F, cap / std::max(bl.second, h + 1))), [&](int nf) {
                             return block_time(dbl, kRingBlue, h, passes, nf, (double)nf * bl.second * bl.first);
                         }));
                }
                return best;
            };
            // the search for the other passes only where Bluestein does not win
            // without them
            kind = fastest(0);
            if (kind != kRingBlue) {
                double rest = 0;
                for (int dir = 0; dir < 2; ++dir) {
                    first[dir] = plan_passes(h, rem, dir == 1, dbl);
                    rest += 0.5 * (first[dir].rad.size() - 1);
                }
                kind = fastest(rest);
            }
            if (kind != kRingConv) lp.conv = PassPlan();
        }
        if (kind != kRingBlue) {
            lp.L = h;
            lp.blue = 0;
        } else {
            lp.L = Lb <= cap ? bl.second : Lb;
            lp.blue = 1;
        }
        if (std::max(lp.L, h + 1) > cap) return SHTX_EUNSUPPORTED;
        // not supported: a register prime of 11 or more with more butterflies
        // than a block has threads
        for (int q : f)
            if (!lp.blue && q >= 11 && lp.L / q > kFftThreads) return SHTX_EUNSUPPORTED;
        for (int dir = 0; dir < 2; ++dir) {
            PassPlan &pp = lp.pass[dir];
            pp = lp.blue ? blues[lp.L].pass[dir] : rem > 1 ? first[dir] : plan_passes(lp.L, 1, dir == 1, dbl);
            const int nconv = (int)lp.conv.rad.size(), P = nconv ? rem - 1 : 0;
            if (nconv && !pp.rad.empty()) {
                pp.rad.erase(pp.rad.begin());
                pp.rad.insert(pp.rad.begin(), lp.conv.rad.begin(), lp.conv.rad.end());
                pp.seam = lp.conv.seam;
            }
            if (pp.rad.empty() || (int)pp.rad.size() > kMaxRadices) return SHTX_EUNSUPPORTED;
            lp.pass_off[dir] = (int)p.passes.size();
            for (int s = 0, Ns = 1; s < (int)pp.rad.size(); ++s) {
                PassDesc q{};
                const int len = s < nconv ? P : lp.L;
                q.R = pp.rad[s];
                q.Ns = Ns;
                q.nbf = len / q.R;
                q.tstep = len / (Ns * q.R);
                q.mg_nbf = div_magic(q.nbf);
                q.mg_ns = div_magic(Ns);
                p.passes.push_back(q);
                Ns = s == pp.seam ? q.R : s == nconv - 1 ? rem : Ns * q.R;  // the seam begins the second FFT
            }
        }
        auto push = [&](long double re, long double im) {
            pool.push_back(re);
            pool.push_back(im);
        };
        auto root = [&](long double a) {  // exp(-i a)
            long double si, co;
            sincosl(a, &si, &co);
            // exact at the quarter turns, where cosl(pi / 2) is 1e-20: values that
            // cancel would keep a residue of that times the others
            push(std::fabs(co) < 1e-18L ? 0.0L : co, std::fabs(si) < 1e-18L ? 0.0L : -si);
        };
        lp.post = (int64_t)pool.size() / 2;
        for (int m = 0; m <= h; ++m) root(2.0L * pi * m / n);
        // roots of unity of L: the second half mirrors the first; a plain ring's
        // first half is every other entry of the n-th roots above, Bluestein
        // lengths are shared between rings
        int64_t &tw = tws[lp.L];
        if (!lp.blue || !tw) {
            tw = (int64_t)pool.size() / 2;
            for (int k = 0; k < lp.L; ++k) {
                const size_t i = 2 * (size_t)(2 * k > lp.L ? tw + lp.L - k : lp.post + 2 * k);
                if (lp.blue && 2 * k <= lp.L) {
                    root(2.0L * pi * k / lp.L);
                } else {
                    const long double re = pool[i], im = pool[i + 1];
                    push(re, 2 * k > lp.L ? -im : im);
                }
            }
        }
        lp.tw = tw;
        lp.chirp = lp.bhat = -1;
        if (!lp.conv.rad.empty()) {
            // roots of unity of P, (g^k, g^-k), and the spectrum over P of the
            // filter W_p^(g^-k), shared between rings
            const int pr = rem, P = pr - 1;
            auto &cv = convs[pr];
            if (!cv[0]) {
                std::vector<int> g((size_t)P);
                const int root0 = primitive_root(pr);
                for (int k = 0, x = 1; k < P; ++k, x = (int)((int64_t)x * root0 % pr)) g[k] = x;
                std::vector<cld> w((size_t)P), b((size_t)P);
                cv[0] = (int64_t)pool.size() / 2;
                for (int k = 0; k < P; ++k) {
                    root(2.0L * pi * k / P);
                    w[k] = {pool[pool.size() - 2], pool[pool.size() - 1]};
                    const long double a = 2.0L * pi * g[(P - k) % P] / pr;
                    b[k] = {cosl(a), -sinl(a)};
                }
                dft_ld(b.data(), P, w, P);
                cv[1] = (int64_t)pool.size() / 2;
                for (int k = 0; k < P; ++k) push(b[k].real() / P, b[k].imag() / P);
                cv[2] = (int64_t)pool.size() / 2;
                const long double bias = dbl ? 0x1p52L : 0x1p23L;
                for (int k = 0; k < P; ++k) push(bias + g[k], bias + g[(P - k) % P]);
            }
            lp.bhat = cv[1];
            lp.conv_tw = cv[0];
            lp.conv_perm = cv[2];
            lp.conv_p = pr;
        }
        if (lp.blue) {
            lp.chirp = (int64_t)pool.size() / 2;
            for (int k = 0; k < h; ++k) {
                int64_t t = ((int64_t)k * k) % (2 * (int64_t)h);
                root(pi * (long double)t / h);
            }
            std::vector<long double> bre, bim;
            bluestein_filter(h, lp.L, &pool[2 * lp.tw], &pool[2 * lp.chirp], bre, bim);
            lp.bhat = (int64_t)pool.size() / 2;
            for (int k = 0; k < lp.L; ++k) push(bre[k], bim[k]);
        }
        lens[n] = lp;
    }
    size_t celem = dbl ? 16 : 8;
    p.twid_elems = (int64_t)pool.size() / 2;
    p.twid_host.assign(pool.begin(), pool.end());
    p.workspace_bytes += (size_t)p.twid_elems * celem;

    p.rings.resize(nlat);
    int64_t goff = 0, foff = 0;
    for (int j = 0; j < nlat; ++j) {
        RingDesc d{};
        const LenPlan &lp = lens[p.nlon[j]];
        d.n = p.nlon[j];
        d.h = d.n / 2;
        d.M = p.cutoff[j];
        d.L = lp.L;
        d.blue = lp.blue;
        d.nrad = (int)lp.pass[0].rad.size();
        d.nrad_r = (int)lp.pass[1].rad.size();
        d.pass_off = lp.pass_off[0];
        d.pass_off_r = lp.pass_off[1];
        d.fuse_in = lp.pass[0].fuse_in;
        d.fuse_out = lp.pass[0].fuse_out;
        d.fuse_in_r = lp.pass[1].fuse_in;
        d.fuse_out_r = lp.pass[1].fuse_out;
        d.seam = lp.pass[0].seam;
        d.seam_r = lp.pass[1].seam;
        d.blue_cost = lp.blue ? (float)blues[lp.L].cost : lp.conv.rad.empty() ? 0.f : (float)lp.conv.cost;
        d.conv = (int)lp.conv.rad.size();
        d.conv_p = lp.conv_p;
        d.conv_tw_off = lp.conv_tw;
        d.conv_perm_off = lp.conv_perm;
        d.lbuf = std::max(d.L, d.h + 1);
        d.lbufp = d.lbuf;
        d.tw_off = lp.tw;
        d.post_off = lp.post;
        d.chirp_off = lp.chirp;
        d.bhat_off = lp.bhat;
        d.grid_off = goff;
        d.four_off = foff;
        d.w = 0.0;  // filled in once the device has computed the weights
        goff += d.n;
        foff += (int64_t)(d.M + 1) * F;
        p.rings[j] = d;
    }
    p.npts = goff;
    p.nfour = foff / F;
    if (p.nfour > INT32_MAX) return SHTX_EUNSUPPORTED;  // ring offsets are stored as int32 / nfld
    int rc = fft_blocking(p, cap);
    if (rc != SHTX_OK) return rc;

    // ---- GEMM work lists ----------------------------------------------------------
    gemm_tiles(prec, trunc, nfld, &p.inv_bm, &p.inv_bn, &p.dir_bm, &p.dir_bn);
    rc = gemm_work_lists(p);
    if (rc != SHTX_OK) return rc;

    p.workspace_bytes += (size_t)p.nfour * F * celem;
    return SHTX_OK;
}

// Full plan: host layout, then the device work (nodes, weights, tables,
// uploads, workspace) on `stream`.
int build_plan(Plan &p, int trunc, int grid, int nlat, int nlon_full, int nfld, int prec,
               unsigned flags, hipStream_t stream)
{
    auto t0 = std::chrono::steady_clock::now();
    int rc = plan_layout(p, trunc, grid, nlat, nlon_full, nfld, prec, flags);
    if (rc != SHTX_OK) return rc;
    if (!gemm_shapes_ok(p) || !fft_shapes_ok(p)) return SHTX_EUNSUPPORTED;
    const int N = trunc, NL = nlat / 2;
    PLAN_TRY(hipGetDevice(&p.device));

    // ---- Gauss nodes and Legendre tables (device, FP64) ---------------------
    PLAN_TRY(hipMalloc(&p.d_mu, sizeof(double) * nlat));
    PLAN_TRY(hipMalloc(&p.d_w, sizeof(double) * nlat));
    PLAN_TRY(launch_gauss_nodes(nlat, p.d_mu, p.d_w, stream));

    PLAN_TRY(hipMalloc(&p.d_tab_inv, table_entry_bytes(p, true) * p.tab_elems));
    PLAN_TRY(hipMalloc(&p.d_tab_dir, table_entry_bytes(p, false) * p.tab_elems));
    PLAN_TRY(hipMalloc(&p.d_diag, sizeof(double) * (size_t)NL * (N + 1)));
    PLAN_TRY(hipMalloc(&p.d_diag_e, sizeof(int) * (size_t)NL * (N + 1)));
    PLAN_TRY(hipMalloc(&p.d_mmax, sizeof(unsigned long long) * (N + 1)));
    PLAN_TRY(upload(&p.d_mb, p.mb));
    PLAN_TRY(launch_legendre_tables(p, stream));
    PLAN_TRY(hipStreamSynchronize(stream));
    // exponents were decided on the device; refresh the host copy
    PLAN_TRY(hipMemcpy(p.mb.data(), p.d_mb, sizeof(MBlock) * p.mb.size(), hipMemcpyDeviceToHost));
    (void)hipFree(p.d_diag);
    p.d_diag = nullptr;
    (void)hipFree(p.d_diag_e);
    p.d_diag_e = nullptr;
    (void)hipFree(p.d_mmax);
    p.d_mmax = nullptr;


    std::vector<double> w(nlat);
    PLAN_TRY(hipMemcpy(w.data(), p.d_w, sizeof(double) * nlat, hipMemcpyDeviceToHost));
    for (int j = 0; j < nlat; ++j) p.rings[j].w = w[j];
    for (int j = 0; j < nlat / 2; ++j) p.qmax = std::max(p.qmax, 0.5 * w[j]);
    if (prec == SHTX_FP16X3) {
        // written by every transform before it is read; zero until then (the
        // autotuner times the GEMMs alone)
        PLAN_TRY(hipMalloc(&p.d_fmax, sizeof(unsigned) * nfld));
        PLAN_TRY(hipMemset(p.d_fmax, 0, sizeof(unsigned) * nfld));
    }

    const bool dbl = prec == SHTX_FP64;
    size_t celem = dbl ? 16 : 8;
    {
        size_t bytes = (size_t)p.twid_elems * celem;
        PLAN_TRY(hipMalloc(&p.d_twid, bytes));
        if (dbl) {
            PLAN_TRY(hipMemcpy(p.d_twid, p.twid_host.data(), bytes, hipMemcpyHostToDevice));
        } else {
            std::vector<float> host(p.twid_host.size());
            for (size_t i = 0; i < host.size(); ++i) host[i] = (float)p.twid_host[i];
            PLAN_TRY(hipMemcpy(p.d_twid, host.data(), bytes, hipMemcpyHostToDevice));
        }
        std::vector<double>().swap(p.twid_host);
    }
    PLAN_TRY(upload(&p.d_rings, p.rings));
    {
        std::vector<int64_t> fo(nlat);
        for (int j = 0; j < nlat; ++j) fo[j] = p.rings[j].four_off;
        PLAN_TRY(upload(&p.d_ring_four_off, fo));
        std::vector<RingPair> rp(nlat / 2);
        for (int j = 0; j < nlat / 2; ++j)
            rp[j] = RingPair{(int)(fo[j] / nfld), (int)(fo[nlat - 1 - j] / nfld)};
        PLAN_TRY(upload(&p.d_ring_pair, rp));
        if (dbl) {
            std::vector<double> q(nlat / 2);
            for (int j = 0; j < nlat / 2; ++j) q[j] = 0.5 * w[j];
            PLAN_TRY(upload(reinterpret_cast<double **>(&p.d_ring_q), q));
        } else {
            std::vector<float> q(nlat / 2);
            for (int j = 0; j < nlat / 2; ++j) q[j] = (float)(0.5 * w[j]);
            PLAN_TRY(upload(reinterpret_cast<float **>(&p.d_ring_q), q));
        }
    }
    PLAN_TRY(upload(&p.d_passes, p.passes));
    // checks every launch shape once more and uploads the work lists
    rc = apply_shapes(p, p.inv_bm, p.inv_bn, p.dir_bm, p.dir_bn, p.fft_cap);
    if (rc != SHTX_OK) return rc;
    PLAN_TRY(fft_prepare(p));
    PLAN_TRY(hipEventCreateWithFlags(&p.done, hipEventDisableTiming));

    PLAN_TRY(hipMalloc(&p.d_four, (size_t)p.nfour * nfld * celem));
    if (flags & SHTX_FLAG_UV) {
        PLAN_TRY(hipMalloc(&p.d_uvspec, (size_t)p.nspec * nfld * celem));
        p.workspace_bytes += (size_t)p.nspec * nfld * celem;
    }

    if (flags & SHTX_FLAG_AUTOTUNE) {
        int trc = autotune_plan(p, stream);
        if (trc != SHTX_OK) return trc;
    }

    if (flags & SHTX_FLAG_TIMING) {
        p.timing_on = true;
        p.ev_start.resize(Plan::kMaxTimed);
        p.ev_stop.resize(Plan::kMaxTimed);
        p.ev_kind.resize(Plan::kMaxTimed);
        for (int i = 0; i < Plan::kMaxTimed; ++i) {
            PLAN_TRY(hipEventCreate(&p.ev_start[i]));
            PLAN_TRY(hipEventCreate(&p.ev_stop[i]));
        }
    }
    PLAN_TRY(hipStreamSynchronize(stream));
    p.plan_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return SHTX_OK;
}

}  // namespace shtx
