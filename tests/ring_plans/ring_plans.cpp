// Ring-FFT plans of the built library, for the host test of what the GPU tests
// reach: for every "precision nlon nfld cap nlat" on standard input (precision 0
// FP64, 1 FP32; cap 0: the default blocking) the plan of a full grid of nlat such
// rings, as words on one line: kind:radix of every pass of both directions
// (kinds as FftPassKind; B before a pass of Bluestein's that is joined to the
// grid), gp:p of a general prime pass and shape:NIxNJ of its work items, residue
// if a root of unity is next to 0 but not 0; or "refused".  With an argument "kernels" instead: the passes and shapes that
// have a kernel.  No GPU.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <set>
#include <string>

#include "shtx_internal.h"

using namespace shtx;

namespace {

std::string word(const char *b, int kind, int radix)
{
    return std::string(b) + std::to_string(kind) + ":" + std::to_string(radix);
}

std::string shape_word(int shape)
{
    return "shape:" + std::to_string(shape / 8) + "x" + std::to_string(shape % 8);
}

void print(const std::set<std::string> &words)
{
    for (const std::string &w : words) std::printf("%s ", w.c_str());
    std::printf("\n");
}

std::set<std::string> kernels(bool dbl)
{
    std::set<std::string> out;
    for (int R = 2; R <= 32; ++R) {
        for (int kind = kPassLds; kind <= kPassScatter; ++kind)
            if (fft_radix_ok(kind, dbl, R)) out.insert(word("", kind, R));
        if (blue_first_radix(R, dbl)) out.insert(word("B", kPassFromGrid, R));
        if (blue_last_radix(R, dbl)) out.insert(word("B", kPassToGrid, R));
    }
#define SHTX_GP(NI, NJ) out.insert(shape_word(gp_shape(NI, NJ)));
    SHTX_GP_SHAPES(SHTX_GP)
#undef SHTX_GP
    return out;
}

void ring_words(const Plan &p, const RingDesc &d, std::set<std::string> &out)
{
    for (int64_t i = 2 * d.post_off; i < 2 * (d.post_off + d.h + 1); ++i)
        if (p.twid_host[i] != 0 && std::fabs(p.twid_host[i]) < 1e-17) out.insert("residue");
    for (int64_t i = 2 * d.tw_off; i < 2 * (d.tw_off + d.L); ++i)
        if (p.twid_host[i] != 0 && std::fabs(p.twid_host[i]) < 1e-17) out.insert("residue");
    for (int dir = 0; dir < 2; ++dir) {
        const int off = dir ? d.pass_off_r : d.pass_off, n = dir ? d.nrad_r : d.nrad;
        const int fin = dir ? d.fuse_in_r : d.fuse_in, fout = dir ? d.fuse_out_r : d.fuse_out;
        const int seam = dir ? d.seam_r : d.seam;
        for (int s = 0; s < n; ++s) {
            const int R = p.passes[off + s].R;
            if (s < d.conv) {
                out.insert(word("", s == 0 ? kPassGather : s == seam ? kPassSubSeam
                                    : s == d.conv - 1                ? kPassScatter
                                                                     : kPassSub, R));
                continue;
            }
            const bool first = s == 0 && fin, last = s == n - 1 && fout;
            if (!first && !last && gp_radix(R, p.prec == SHTX_FP64)) {
                out.insert("gp:" + std::to_string(R));
                continue;
            }
            const int kind = d.blue && s == seam ? kPassSeam
                             : first             ? (dir ? kPassFromGrid : kPassFromFour)
                             : last              ? (dir ? kPassToFour : kPassToGrid)
                                                 : kPassLds;
            out.insert(word(d.blue && (first || last) ? "B" : "", kind, R));
        }
    }
}

}  // namespace

int main(int argc, char **argv)
{
    if (argc > 1 && !std::strcmp(argv[1], "kernels")) {
        print(kernels(true));
        print(kernels(false));
        return 0;
    }
    int prec, nlon, nfld, cap, nlat;
    while (std::scanf("%d %d %d %d %d", &prec, &nlon, &nfld, &cap, &nlat) == 5) {
        Plan p;
        const int trunc = nlon > 40 ? 20 : (nlon - 1) / 2;
        if (plan_layout(p, trunc, SHTX_GRID_FULL, nlat, nlon, nfld, prec, 0) != SHTX_OK ||
            (cap && fft_blocking(p, cap) != SHTX_OK) || !fft_shapes_ok(p)) {
            std::printf("refused\n");
            continue;
        }
        std::set<std::string> out;
        ring_words(p, p.rings[0], out);
        for (const FftItem &it : p.fft_items)
            if (it.ring >= 0 && it.shape) out.insert(shape_word(it.shape));
        print(out);
    }
    return 0;
}
