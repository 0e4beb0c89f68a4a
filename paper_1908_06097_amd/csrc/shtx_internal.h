// Internal declarations shared by the plan code and the HIP kernels of libshtx.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "../../include/shtx.h"

namespace shtx {

// Legendre tables pad both the ring and the parity-k dimension of every m
// block to a multiple of this, so that GEMM tiles (whose sizes divide it)
// always read inside the block.
constexpr int kTablePad = 128;

// Ring-FFT kernels hold at most this many complex values of one block in LDS.
constexpr int kFftCapF32 = 8192;  // 64 KiB: two blocks per CU with the prime-pass roots
constexpr int kFftCapF64 = 8192;  // 128 KiB: one block per CU (the FP64 passes use 228 VGPRs)
constexpr int kFftThreads = 512;

// Butterflies per thread in an in-place radix-R Stockham pass (rounds of
// kFftThreads): enough for a block's cap complex values, but one round from
// radix 13 on (a second would spill), to which the blocking keeps a block's
// fields.
__host__ __device__ constexpr int fft_rounds(int cap, int R)
{
    return R >= 13 ? 1 : (cap / R + kFftThreads - 1) / kFftThreads;
}

// Kinds of Stockham pass, by where the pass reads and writes: LDS to LDS in
// place; the r2c kernel's first pass, from the grid row; the c2r kernel's first
// pass, from the Fourier rows with the merge step; the c2r kernel's last pass,
// to the grid row; the r2c kernel's last pass, with the split step to the
// Fourier rows; the seam between Bluestein's two FFTs, in LDS; and of a prime
// pass by convolution, all in LDS, its first pass, those between, its seam and
// its last pass.
enum FftPassKind {
    kPassLds = 0,
    kPassFromGrid = 1,
    kPassFromFour = 2,
    kPassToGrid = 3,
    kPassToFour = 4,
    kPassSeam = 5,
    kPassGather = 6,
    kPassSub = 7,
    kPassSubSeam = 8,
    kPassScatter = 9
};

constexpr int kTopRadix = 23;  // of any kind

// Radices with a butterfly of each kind.  The Fourier-side passes hold a pair of
// butterflies (j and its mirror) per thread, so their radices stop earlier;
// FP64 values take twice the registers.  The sets end where the butterfly would
// spill at the two blocks (FP64: one) per CU that the LDS allows, and hold no
// radix that no ring's cheapest passes have.
__host__ __device__ constexpr bool fft_radix_ok(int kind, bool dbl, int R)
{
    if (R < 2) return false;
    switch (kind) {
    case kPassLds: return R <= 13 || R == 16 || R == 17 || (!dbl && (R == 18 || R == 19 || R == 23));
    case kPassFromGrid: return (R <= 13 && R > (dbl ? 2 : 1)) || R == 16 || (!dbl && (R == 15 || R == 17 || R == 18));
    case kPassFromFour: return dbl ? R > 2 && R <= 9 : R <= 10;
    case kPassToGrid: return R <= 10 || R == 12 || R == 16 || (!dbl && (R == 14 || R == 15 || R == 18 || R == 20));
    case kPassToFour: return R <= 6 || R == 8 || (!dbl && (R == 7 || R == 9));
    case kPassSeam: return R == 9 || R == 10 || (dbl ? R == 12 : R == 15 || R == 18);
    case kPassGather: return R == 3 || (R > 4 && R <= 19) || R == 23;
    case kPassSub: return R <= 19 || R == 23;
    case kPassScatter: return R <= 11 || (R >= 13 && R <= 17) || R == 19;
    case kPassSubSeam:
        return R == 4 || R == 6 || R == 8 || R == 9 || R == 10 || (R >= 14 && R <= 16) || (!dbl && (R == 12 || R == 18));
    }
    return false;
}
// First radices of Bluestein's first FFT that read the grid themselves (with
// the chirp), and last ones of its second that write it.
__host__ __device__ constexpr bool blue_first_radix(int R, bool dbl)
{
    return R == 9 || R == 10 || R == 12 || (dbl ? R == 8 : R == 15 || R == 18);
}
__host__ __device__ constexpr bool blue_last_radix(int R, bool dbl)
{
    return R == 8 || R == 9 || R == 10 || (dbl ? R == 4 : R == 12 || R == 16);
}

// General prime pass: a ring whose half-length has one prime factor p above
// the register radices, p <= kGpMaxPrime, may run it as the first pass on the
// matrix cores (the plan chooses between it, a convolution and Bluestein),
// reading the p-th roots of unity from p LDS entries after the
// field slots.  Its outputs come in units of 16 rows t (t = 0 .. (p-1)/2) by
// 16 columns (butterfly, real | imaginary part); each wave holds one tile of
// NI x NJ of them, at most kGpUnits (more would push the FFT kernels past the
// registers that keep two blocks, FP64 one, per CU).
constexpr int kGpMaxPrime = 1021;
constexpr int kGpUnits = 6;
constexpr int kGpFieldUnits = 32;  // and one field at most this many in all
__host__ __device__ constexpr int gp_row_tiles(int p) { return ((p - 1) / 2 + 16) / 16; }
__host__ __device__ constexpr int gp_col_tiles(int nbutterflies) { return (2 * nbutterflies + 15) / 16; }
__host__ __device__ constexpr int gp_shape(int ni, int nj) { return 8 * ni + nj; }
// Tile shapes with an instantiation (X(NI, NJ)).
#define SHTX_GP_SHAPES(X) \
    X(1, 1) X(1, 2) X(2, 1) X(1, 3) X(3, 1) X(2, 2) X(1, 4) X(4, 1) X(1, 5) X(5, 1) X(2, 3) X(3, 2)
// Whether one tile of a shape per wave covers the units of nb butterflies.
inline bool gp_shape_ok(int shape, int p, int nb)
{
    const int ni = shape / 8, nj = shape % 8;
    if (ni < 1 || nj < 1 || ni * nj > kGpUnits) return false;
    return (gp_row_tiles(p) + ni - 1) / ni * ((gp_col_tiles(nb) + nj - 1) / nj) <= kFftThreads / 64;
}
// The cheapest shape that does, 0 if none: MFMAs by the units of a wave, LDS
// reads by its row tiles (root reads, with bank conflicts) and column tiles.
inline double gp_cost(int shape)
{
    const int ni = shape / 8, nj = shape % 8;
    return ni * nj + 0.25 * ni + 0.125 * nj;
}
inline int gp_best_shape(int p, int nb)
{
    int best = 0;
#define SHTX_GP(NI, NJ)                                                                       \
    if (gp_shape_ok(gp_shape(NI, NJ), p, nb) && (!best || gp_cost(gp_shape(NI, NJ)) < gp_cost(best))) \
        best = gp_shape(NI, NJ);
    SHTX_GP_SHAPES(SHTX_GP)
#undef SHTX_GP
    return best;
}
constexpr int kMaxRadices = 12;
// Primes above the register butterflies run as general prime passes.
__host__ __device__ constexpr bool gp_radix(int R, bool dbl) { return R > kTopRadix || (dbl && (R == 19 || R == 23)); }

// One m block of the Legendre tables.
struct MBlock {
    int R;          // northern rings carrying m (M_j >= m): j0 .. j0 + R - 1
    int j0;         // first such ring
    int K0, K1;     // number of n = m + p + 2k <= N for parity p = 0, 1
    int Rp, Kp;     // padded ring and parity-k extents
    int e;          // power-of-two exponent applied to the stored pieces or units
    int pad_;
    int64_t off;    // entries of the m blocks before this one (2 Kp Rp each)
};

// One GEMM work item: wavenumber m, row tile, column tile (m < 0: no work).
struct GemmItem {
    int m, tr, tc, pad_;
};

// One ring of the grid (device copy of the FFT plan for that ring).
struct RingDesc {
    int n;        // ring length (even)
    int h;        // n / 2: length of the complex FFT
    int M;        // ring cutoff
    int L;        // executed FFT length (h, or the Bluestein length >= 2h - 1)
    int nrad, nrad_r;  // number of Stockham passes, c2r and r2c
    int blue;     // 1 if the length-h DFT goes through Bluestein's convolution
    int fb;       // fields per FFT block for this ring
    int lbuf;     // complex values per field slot: max(L, h + 1)
    int lbufp;    // LDS entries per field slot
    int pass_off, pass_off_r;  // first PassDesc of the c2r and the r2c passes
    int fuse_in, fuse_out;      // c2r: first pass merges, last pass writes the grid
    int fuse_in_r, fuse_out_r;  // r2c: first pass reads the grid, last pass splits
    int seam, seam_r;           // index of Bluestein's seam pass, c2r and r2c (-1: none)
    float blue_cost;            // cost of Bluestein's or the convolution's passes (host only)
    int conv, conv_p;           // a prime pass by convolution: its passes (0: none), its prime
    int64_t conv_tw_off;        // W_{p-1}
    int64_t conv_perm_off;      // (g^k, g^-k) mod p, g a primitive root, k < p - 1, each plus 2^23 (FP64: 2^52)
    int64_t tw_off;     // W_L[k] = exp(-2 pi i k / L), k < L
    int64_t post_off;   // exp(-2 pi i m / n), m <= h
    int64_t chirp_off;  // Bluestein chirp exp(-pi i k^2 / h), k < h
    int64_t bhat_off;   // Bluestein filter spectrum / L, L entries; a convolution's / (p - 1), p - 1 entries
    int64_t grid_off;   // first point of the ring inside one grid field
    int64_t four_off;   // first complex of the ring's [m][nfld] block
    double w;           // Gauss weight
};

// One Stockham pass of a ring length's FFT (shared by every ring of that
// length).  Divisions by nbf and Ns are done as mul_hi(a, magic) with
// magic = ceil(2^32 / d), exact for a * d < 2^32 (magic 0 stands for d = 1).
struct PassDesc {
    int R;          // radix
    int Ns;         // product of the radices of the earlier passes
    int nbf;        // butterflies per field: L / R
    int tstep;      // twiddle table stride of the butterfly index: L / (Ns R)
    unsigned mg_nbf, mg_ns;
};

__host__ __device__ inline unsigned div_magic(int d) { return d <= 1 ? 0u : 0xFFFFFFFFu / (unsigned)d + 1u; }

// Fourier-workspace offsets of a northern ring and its southern mirror, in
// units of nfld complex values (RingDesc::four_off / nfld).
struct __attribute__((aligned(8))) RingPair {
    int n, s;
};

// One FFT work item: a ring, a run of fields (ring < 0: no work) and the tile
// shape of the ring's prime pass for them, if it has one.
struct FftItem {
    int ring, f0, nf, shape;
};

enum TransformKind { kInverse = 0, kDirect = 1, kInverseAdj = 2, kDirectAdj = 3, kWind = 4 };
constexpr int kKinds = 5;

// The split-precision forms: hi + lo halves of bfloat16 or IEEE half.
inline bool split_form(int prec) { return prec == SHTX_BF16X3 || prec == SHTX_FP16X3; }
// 16-bit pieces of an operand in the half-precision matrix-core GEMM (FP32: three
// bfloat16).
__host__ __device__ constexpr int split_pieces(int prec) { return prec == SHTX_FP32 ? 3 : 2; }
// Scale of a single-precision plan's table units: the last bit of the smallest
// normal float, 2^-149, times 2^16 is bfloat16's smallest value.
constexpr int kF32TableExp = 16;
constexpr float kF32TableScale = 65536.f;

struct Plan {
    int trunc = 0, grid = 0, nlat = 0, nlon_full = 0, nfld = 0, prec = 0;
    unsigned flags = 0;
    int64_t nspec = 0, npts = 0, nfour = 0;
    std::vector<int32_t> nlon;
    std::vector<int> cutoff;
    std::vector<MBlock> mb;
    std::vector<RingDesc> rings;
    int max_nlon = 0;

    // GEMM tiling chosen at plan time (depends on precision).
    int inv_bm = 0, inv_bn = 0, dir_bm = 0, dir_bn = 0;
    // Column fragments of the few-fields GEMM (gemm_narrow), 0: tiles as above.
    int inv_narrow = 0, dir_narrow = 0;
    std::vector<GemmItem> inv_items, dir_items;
    std::vector<FftItem> fft_items;
    std::vector<PassDesc> passes;
    int fft_lds_bytes = 0;
    int fft_lds_max = 0;  // complex entries of LDS the largest FFT block may use
    int fft_cap = 0;      // LDS complex values per FFT block the blocking was made for
    int tuned = 0;        // 0 default tiles, 1 timed by the autotuner, 2 from the tune cache
    // True once every kernel's work list and launch shape has passed the host
    // checks and the device copies of the lists match them; launches check
    // only this flag, so the per-item checks run at plan time, not per call.
    bool shapes_ok = false;
    int device = -1;              // HIP device the plan's memory lives on
    hipEvent_t done = nullptr;    // recorded after each transform's launches
    bool timing_on = false;       // record kernel events (plans made with SHTX_FLAG_TIMING)

    // Device memory.
    double *d_mu = nullptr, *d_w = nullptr;  // nlat
    double *d_diag = nullptr;                // [NL][N+1] sectoral seeds q (plan time only) ...
    int *d_diag_e = nullptr;                 // ... and their exponents E: P̄_m^m = q 2^E
    // Legendre tables of the inverse- and the direct-shaped GEMM (TableLayout).
    void *d_tab_inv = nullptr, *d_tab_dir = nullptr;
    unsigned long long *d_mmax = nullptr;                  // per-m max |P̄| bits (plan time)
    MBlock *d_mb = nullptr;
    GemmItem *d_inv_items = nullptr, *d_dir_items = nullptr;
    RingDesc *d_rings = nullptr;
    int64_t *d_ring_four_off = nullptr;  // per ring: RingDesc::four_off
    RingPair *d_ring_pair = nullptr;     // per northern ring
    void *d_ring_q = nullptr;            // per northern ring: w_j / 2 in grid precision
    FftItem *d_fft_items = nullptr;
    PassDesc *d_passes = nullptr;
    void *d_twid = nullptr;  // FFT twiddle pool (complex, grid precision)
    int64_t twid_elems = 0;  // complex entries in the pool
    std::vector<double> twid_host;  // pool (re, im) before upload
    void *d_four = nullptr;  // Fourier workspace [ring][m][nfld] complex
    // SHTX_FP16X3: per field, the largest magnitude (float bits) of the data
    // the next Legendre GEMM splits (spectral input or Fourier workspace)
    unsigned *d_fmax = nullptr;
    // SHTX_FLAG_UV: spectral wind images [nfld][nspec] (U then V) between the
    // wind step and the inverse transform
    void *d_uvspec = nullptr;
    double qmax = 0.0;  // max over northern rings of w_j / 2
    int64_t tab_elems = 0;   // elements per table layout
    size_t table_bytes = 0, workspace_bytes = 0;
    double legendre_flops = 0.0;
    double plan_seconds = 0.0;

    // Graph cache (one per transform kind, keyed on pointers and stream).
    struct GraphEntry {
        hipGraphExec_t exec = nullptr;
        const void *in = nullptr, *in2 = nullptr;
        void *out = nullptr;
        hipStream_t stream = nullptr;
    } graphs[kKinds];

    // Kernel timing.
    static constexpr int kMaxTimed = 4096;
    std::vector<hipEvent_t> ev_start, ev_stop;
    std::vector<int> ev_kind;
    int n_timed = 0;
};

// Element sizes.
inline int grid_elem_bytes(int prec) { return prec == SHTX_FP64 ? 8 : 4; }

// Transform-call helpers of the C ABI (capi.cpp): argument checks (SHTX_OK or
// SHTX_EINVAL, nothing launched), and the per-plan completion event.
int check_args(const Plan &p, int kind, const void *in, const void *out, const void *in2 = nullptr);
hipError_t mark_done(Plan &p, hipStream_t s);
hipError_t wait_done(Plan &p);

// Kernel launchers (each checks its launch shape on the host first).
hipError_t launch_gauss_nodes(int nlat, double *mu, double *w, hipStream_t s);
hipError_t launch_legendre_tables(Plan &p, hipStream_t s);
// `fmax` is the per-field maxima buffer of a SHTX_FP16X3 plan (nfld words;
// ignored by the other forms): the plan's own, or a caller-provided one.
hipError_t launch_gemm_inverse(const Plan &p, const void *spec, void *four, unsigned *fmax, hipStream_t s);
hipError_t launch_gemm_direct(const Plan &p, const void *four, void *spec, bool adjoint, unsigned *fmax,
                              hipStream_t s);
hipError_t launch_fft_c2r(const Plan &p, const void *four, void *grid, bool adjoint,
                          hipStream_t s);
hipError_t launch_fft_r2c(const Plan &p, const void *grid, void *four, bool adjoint, unsigned *fmax,
                          hipStream_t s);
// Wind step of shtx_uv_trans: spectral vorticity and divergence of truncation
// trunc - 1 (nfld / 2 fields each) -> spectral U and V of truncation trunc.
hipError_t launch_uv_spec(const Plan &p, const void *vor, const void *dvg, void *out, hipStream_t s);
// Fields per ring-FFT block are at most this many when the r2c kernel also
// records each field's largest output magnitude (SHTX_FP16X3 plans).
constexpr int kFmaxFields = 1024;

// Host checks that every kernel's work list and launch shape stay inside the
// plan's arrays and the kernels' compile-time limits (no device access).
bool gemm_shapes_ok(const Plan &p);
bool fft_shapes_ok(const Plan &p);
int plan_layout(Plan &p, int trunc, int grid, int nlat, int nlon_full, int nfld, int prec, unsigned flags);

// GEMM tile sizes per precision (rows, columns) for each direction: the
// defaults, and whether a kernel instantiation exists for a shape.
void gemm_tiles(int prec, int trunc, int nfld, int *inv_bm, int *inv_bn, int *dir_bm, int *dir_bn);
bool gemm_tile_supported(int prec, int bm, int bn);
// Few fields: column fragments of the kernel that serves them, whatever the
// tile shapes are (0: the tiled kernels do), and its row tile.
int gemm_narrow(int prec, int nfld, bool inverse);
// How a direction's table is laid out, per m block (inverse | direct):
//   kTabPlain   values of the plan's precision [p][k][r] | [p][r][k], where a
//               kernel of that precision reads them (FP64, few fields)
//   kTabPieces  the split forms: 16-bit pieces [piece][p][k / 8][r][k % 8] |
//               [piece][p][r / 8][k][r % 8]
//   kTabUnits   single precision: floats, times kF32TableScale, in the same order,
//               [p][k / 8][r][k % 8] | [p][r / 8][k][r % 8]; the GEMM cuts them
//               into pieces (stored in pieces they take half as much memory
//               again and gain 2 to 4 % of the direct GEMM and nothing of the
//               inverse, T1279 11.3 against 11.6 ms and 9.9 each)
enum TableLayout { kTabPlain, kTabPieces, kTabUnits };
inline TableLayout table_layout(const Plan &p, bool inverse)
{
    if (p.prec == SHTX_FP64 || (inverse ? p.inv_narrow : p.dir_narrow)) return kTabPlain;
    return p.prec == SHTX_FP32 ? kTabUnits : kTabPieces;
}
inline size_t table_entry_bytes(const Plan &p, bool inverse)
{
    return table_layout(p, inverse) == kTabPieces ? 2 * split_pieces(p.prec) : p.prec == SHTX_FP64 ? 8 : 4;
}
constexpr int kNarrowRows = 64;
// Candidate shapes the autotuner times (count returned, shapes in bm[], bn[]).
int gemm_tile_candidates(int prec, int *bm, int *bn, int max);

// Rebuild the FFT blocking (fields per block within `cap` LDS complex
// values) and the GEMM work lists for the plan's current tile shapes.
int fft_blocking(Plan &p, int cap);
int gemm_work_lists(Plan &p);

// Time the candidate GEMM tile shapes and FFT blockings on this plan and keep
// the fastest (or take them from the tune cache); uploads the work lists.
int autotune_plan(Plan &p, hipStream_t s);
// Set the GEMM tile shapes and FFT blocking of a built plan: rebuilds the
// work lists, checks every launch shape, uploads the lists into new device
// buffers and only then replaces the plan's (the caller makes sure no
// transform is in flight).  On any error the plan is left as it was.
int apply_shapes(Plan &p, int inv_bm, int inv_bn, int dir_bm, int dir_bn, int fft_cap);
// Let the ring-FFT kernels of the plan's precision use the whole LDS of a
// workgroup as dynamic LDS (set per device at plan creation).
hipError_t fft_prepare(const Plan &p);

// Work lists are laid out as 8 equal segments, one per XCD (the hardware
// deals workgroups to the 8 XCDs round-robin), padded with no-op items.
// xcd_remap maps the hardware block index to the item index so that segment x
// runs on XCD x in order: items that share data (the tiles of one m, the field
// runs of one ring) are put in the same segment and share that XCD's L2.
constexpr int kXcds = 8;

__device__ inline int xcd_remap(int bid, int grid)
{
    int per = grid / kXcds;
    return (bid % kXcds) * per + bid / kXcds;
}

// Host helper: place groups of items (each group kept on one XCD) into the 8
// segments, heaviest group first onto the least-loaded segment, and pad.
template <class Item>
std::vector<Item> layout_by_xcd(const std::vector<std::vector<Item>> &groups,
                                const std::vector<double> &cost, const Item &noop)
{
    std::vector<size_t> order(groups.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = i;
    std::sort(order.begin(), order.end(), [&](size_t a, size_t b) { return cost[a] > cost[b]; });
    std::vector<std::vector<Item>> seg(kXcds);
    double load[kXcds] = {0};
    for (size_t g : order) {
        int best = 0;
        for (int x = 1; x < kXcds; ++x)
            if (load[x] < load[best]) best = x;
        load[best] += cost[g];
        seg[best].insert(seg[best].end(), groups[g].begin(), groups[g].end());
    }
    size_t per = 0;
    for (auto &v : seg) per = std::max(per, v.size());
    if (per == 0) per = 1;
    std::vector<Item> out(per * kXcds, noop);
    for (int x = 0; x < kXcds; ++x)
        std::copy(seg[x].begin(), seg[x].end(), out.begin() + x * per);
    return out;
}

}  // namespace shtx

// The opaque handle of the C ABI.
struct shtx_plan_s {
    shtx::Plan p;
};
