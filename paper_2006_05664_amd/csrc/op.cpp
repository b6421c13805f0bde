// Operator descriptors, configuration spaces and the configuration decoder.
#include "op.hpp"

#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <new>
#include <numeric>
#include <sstream>

using namespace opevo;

static const int kMaxThreads = 1024;            // threads per workgroup on gfx950
static const int kMaxLds = 160 * 1024;          // LDS bytes per workgroup on gfx950
static const int64_t kMaxDldsBody = 256;        // unrolled K-loop body of the direct-to-LDS template, instructions
static const int64_t kMaxDldsBody16 = 400;      // the same for members on 16x16x32 atoms
static const int kMaxAcc = 256;                 // fp32 accumulators per lane kept in registers
static const int kPad = 8;                      // LDS row padding of the MFMA template (elements)

int64_t opevo_op::a_elems() const
{
    return kind == OPEVO_CONV2D ? M * K : batch * M * K;   // conv: kernel tensor [Cout][Cin*Hk*Wk]
}

int64_t opevo_op::b_elems() const
{
    return kind == OPEVO_CONV2D ? nimg * cin * hin * win : batch * K * N;
}

namespace opevo {

static opevo_param_desc factor(const char *name, int64_t C, int nu)
{
    opevo_param_desc d;
    std::memset(&d, 0, sizeof d);
    d.type = OPEVO_FACTOR; d.C = C; d.nu = nu; d.name = name;
    return d;
}

static const double kGroupValues[] = {1, 2, 4, 8, 16};
static const int kNumGroupValues = 5;
static const double kUnrollSteps[] = {1, 2, 4, 8};
static const int kNumUnrollSteps = 4;
static const double kReductionWaves[] = {1, 2, 4, 8};
static const int kNumReductionWaves = 4;

static opevo_param_desc permutation(const char *name, int n)
{
    opevo_param_desc d;
    std::memset(&d, 0, sizeof d);
    d.type = OPEVO_PERMUTATION; d.n_values = n; d.name = name;
    return d;
}

static opevo_param_desc discrete(const char *name, const double *values, int n)
{
    opevo_param_desc d;
    std::memset(&d, 0, sizeof d);
    d.type = OPEVO_DISCRETE; d.n_values = n; d.values = values; d.name = name;
    return d;
}

static opevo_param_desc flag(const char *name)
{
    opevo_param_desc d;
    std::memset(&d, 0, sizeof d);
    d.type = OPEVO_CATEGORICAL; d.n_values = 2; d.name = name;
    return d;
}

int op_param_descs(const opevo_op &op, int variant, std::vector<opevo_param_desc> &descs)
{
    descs.clear();
    if (variant == OPEVO_TILE2) {
        if (op.kind != OPEVO_MATMUL) return fail(OPEVO_E_ARG, "the two-level space exists for MatMul only");
        descs = {factor("M", op.M, 2), factor("N", op.N, 2), factor("K", op.K, 2)};
        return OPEVO_OK;
    }
    if (variant == OPEVO_TILE4P) {
        // App. B.3: C_out, H_out, W_out in four factors, C_in, H_k, W_k in two factors each, the binary
        // choice of an explicit unroll and the discrete bound on the unrolled steps; the batch
        // split is kept from the four-level space
        if (op.kind != OPEVO_CONV2D) return fail(OPEVO_E_ARG, "the separately split reduction space exists for Conv2d only");
        descs = {factor("B", op.nimg, 2), factor("Cout", op.M, 4), factor("H", op.hout, 4), factor("W", op.wout, 4),
                 factor("Cin", op.cin, 2), factor("Hk", op.hk, 2), factor("Wk", op.wk, 2), flag("unroll"),
                 discrete("unroll_steps", kUnrollSteps, kNumUnrollSteps)};
        return OPEVO_OK;
    }
    if (variant == OPEVO_TILE4K) {
        // MatMul with the reduction axis in three factors, as App. B.1 splits it; the outermost one is
        // the number of workgroups that share an output tile, each reducing its own part of K
        if (op.kind != OPEVO_MATMUL) return fail(OPEVO_E_ARG, "the split-reduction space exists for MatMul only");
        descs = {factor("M", op.M, 4), factor("N", op.N, 4), factor("K", op.K, 3), flag("unroll")};
        return OPEVO_OK;
    }
    if (variant == OPEVO_TILE4T) {
        // MatMul with the layout of the second operand as a second binary choice: as stored ([K][N]) or
        // transposed to [N][K] by a pre-pass before every launch
        if (op.kind != OPEVO_MATMUL) return fail(OPEVO_E_ARG, "the space with a packed second operand exists for MatMul only");
        descs = {factor("M", op.M, 4), factor("N", op.N, 4), factor("K", op.K, 2), flag("unroll"), flag("bpack")};
        return OPEVO_OK;
    }
    if (variant == OPEVO_TILE4A) {
        // MatMul with the MFMA atom of direct-to-LDS members as a second binary choice: 32x32x16 or 16x16x32
        if (op.kind != OPEVO_MATMUL) return fail(OPEVO_E_ARG, "the space with a choice of MFMA atom exists for MatMul only");
        descs = {factor("M", op.M, 4), factor("N", op.N, 4), factor("K", op.K, 2), flag("unroll"), flag("atom")};
        return OPEVO_OK;
    }
    if (variant == OPEVO_TILE4C) {
        // Conv2d with the fused reduction axis in three factors (partitions along grid z, steps, LDS
        // tile) and the operand layout as a second binary choice
        if (op.kind != OPEVO_CONV2D) return fail(OPEVO_E_ARG, "the split-reduction / channels-last space exists for Conv2d only");
        descs = {factor("B", op.nimg, 2), factor("Cout", op.M, 4), factor("H", op.hout, 4), factor("W", op.wout, 4),
                 factor("R", op.K, 3), flag("unroll"), flag("layout")};
        return OPEVO_OK;
    }
    if (variant == OPEVO_TILE4L) {
        // Conv2d with the input channels in two factors (slabs, channels per slab; every slab holds all the
        // taps) and a three-way choice of how the operands reach the matrix units: gathered from the NCHW
        // image value by value, channels-last copies written by a pre-pass, or an LDS-resident image patch
        // filled straight from the NCHW image; for the last, the number of waves that share a wave tile and split
        // the reduction steps of every slab among themselves
        if (op.kind != OPEVO_CONV2D) return fail(OPEVO_E_ARG, "the space with an LDS-resident image patch exists for Conv2d only");
        descs = {factor("B", op.nimg, 2), factor("Cout", op.M, 4), factor("H", op.hout, 4), factor("W", op.wout, 4),
                 factor("Cin", op.cin, 2), flag("unroll"), flag("layout"), discrete("kwaves", kReductionWaves, kNumReductionWaves)};
        descs[descs.size() - 2].n_values = 3;
        return OPEVO_OK;
    }
    if (variant != OPEVO_TILE4 && variant != OPEVO_TILE4X) return fail(OPEVO_E_ARG, "unknown variant %d", variant);
    switch (op.kind) {
    case OPEVO_MATMUL:
        descs = {factor("M", op.M, 4), factor("N", op.N, 4), factor("K", op.K, 2), flag("unroll")};
        break;
    case OPEVO_BMM:
        descs = {factor("B", op.batch, 2), factor("M", op.M, 4), factor("N", op.N, 4),
                 factor("K", op.K, 2), flag("lds")};
        break;
    case OPEVO_CONV2D:
        descs = {factor("B", op.nimg, 2), factor("Cout", op.M, 4), factor("H", op.hout, 4),
                 factor("W", op.wout, 4), factor("R", op.K, 2), flag("unroll")};
        break;
    default:
        return fail(OPEVO_E_ARG, "unknown operator kind %d", op.kind);
    }
    if (variant == OPEVO_TILE4X) {
        // the order in which a one-dimensional launch walks the grid axes (N tiles, M tiles and,
        // for BMM, batch blocks; first = fastest), and the width of the groups of second-axis
        // tiles it walks together
        descs.push_back(permutation("order", op.kind == OPEVO_BMM ? 3 : 2));
        descs.push_back(discrete("group", kGroupValues, kNumGroupValues));
    }
    return OPEVO_OK;
}

// Row pitch and per-image pitch (in pixels) of the LDS-resident patch for a box of bh x bw output pixels:
// (bh-1)*stride + hk rows of (bw-1)*stride + wk pixels.  padded (unit stride only): the row pitch and the image
// pitch are raised to be congruent to bw and to bh*bw modulo 16, so that consecutive output pixels of the
// flattened box read consecutive groups of LDS banks.
static void patch_pitches(const opevo_op &op, int64_t bh, int64_t bw, bool padded, int64_t &row, int64_t &image)
{
    const int64_t ph = (bh - 1) * op.stride + op.hk, pw = (bw - 1) * op.stride + op.wk;
    row = pw; image = ph * pw;
    if (!padded || op.stride != 1) return;
    row = pw + ((bw - pw) % 16 + 16) % 16;
    image = ph * row + ((bh * bw - ph * row) % 16 + 16) % 16;
}

// How the ragged MFMA template runs a tile of bm x bn with slabs of about bk: wave grid, atoms per wave, slab width.
struct Ragged { int wm = 0, wn = 0, mi = 0, ni = 0, ks = 0, slabs = 0, stages = 1, depth = 1, keep = 0, min_waves = 1; int64_t lds = 0; };

static bool plan_ragged(const opevo_op &op, int64_t bm, int64_t bn, int64_t bk, int64_t kpart, int64_t wgs, bool pipelined, Ragged &out)
{
    // every operand is loaded in pieces of 8 consecutive elements of a row, with 32-bit element offsets inside a batch
    if (kpart < 8 || op.N < 8 || (op.trans_a && op.M < 8) || op.M * op.K >= (int64_t(1) << 31) || op.K * op.N >= (int64_t(1) << 31)) return false;
    const int64_t ma = (bm + 15) / 16, na = (bn + 15) / 16;
    if (ma * na * 256 > 8 * bm * bn || ma * na > 16 * 32) return false;
    const int64_t top = std::max<int64_t>(32, std::min<int64_t>(128, (std::min(bk, kpart) + 31) / 32 * 32));
    // staging registers of a lane with slabs of ks and nt threads
    auto staging = [&](int64_t ks, int64_t nt) {
        const int64_t a_pieces = op.trans_a ? ks * ((bm + 7) / 8) : bm * (ks / 8), b_pieces = ks * ((bn + 7) / 8);
        return 4 * ((a_pieces + nt - 1) / nt + (b_pieces + nt - 1) / nt);
    };
    // Registers: staging and accumulators within 256 with up to eight waves (one or two a SIMD: of 300 compiled members none spilled).
    // With more a lane has 170 (9 - 12 waves) or 128, and what the kernel needs beside staging, accumulators and fragments
    // counts: members with as little as 62 to spare spilled, so 66 are kept free.
    auto room = [&](int64_t ks, int64_t nw, int64_t mi, int64_t ni) {
        const int64_t held = staging(ks, 64 * nw) + 4 * mi * ni;
        return nw <= 8 ? held <= 256 : held + 4 * (mi + ni) + 66 <= 512 / ((nw + 3) / 4);
    };
    // waves: the division with the fewest padded atoms, then the one closest to four waves (one per SIMD; eight where the
    // tile has 64 atoms and more), then the one with the fewest fragment reads
    const int64_t want = ma * na >= 64 ? 8 : 4;
    int64_t best = INT64_MAX;
    for (int64_t wm = 1; wm <= std::min<int64_t>(ma, 16); ++wm)
        for (int64_t wn = 1; wn <= std::min<int64_t>(na, 16 / wm); ++wn) {
            const int64_t mi = (ma + wm - 1) / wm, ni = (na + wn - 1) / wn, nw = wm * wn;
            if (mi * ni > 32 || (nw > 8 && !room(32, nw, mi, ni))) continue;
            const int64_t off = nw > want ? nw - want : (want - nw) * 4;      // too few waves are worse than too many
            const int64_t score = (wm * mi * wn * ni * 8 + off * std::min<int64_t>(ma * na, 32)) * 64 + nw * (mi + ni);
            if (score < best) { best = score; out.wm = int(wm); out.wn = int(wn); out.mi = int(mi); out.ni = int(ni); }
        }
    if (best == INT64_MAX) return false;
    // slab: the member's, rounded up to whole MFMA steps of 32 and at most 128; among the shorter ones the one that pads
    // the reduction least (a slab costs about as much as 8 steps of padding), as far as LDS and staging registers go
    best = INT64_MAX;
    for (int64_t ks = 32; ks <= top; ks += 32) {
        auto odd16 = [](int64_t n) { return ((n + 15) / 16 | 1) * 16; };
        const int64_t slabs = (kpart + ks - 1) / ks;
        const int64_t a_stage = op.trans_a ? ks * odd16(out.wm * out.mi * 16) + ks / 8 * 64 : out.wm * out.mi * 16 * (ks + 8);
        const int64_t b_stage = ks * odd16(out.wn * out.ni * 16) + ks / 8 * 64;
        const int stages = pipelined && slabs > 1 ? 2 : 1;
        const int64_t lds = stages * (a_stage + b_stage) * 2;
        if (lds > kMaxLds || !room(ks, out.wm * out.wn, out.mi, out.ni)) continue;
        const int64_t score = slabs * (ks + 8) + (lds > kMaxLds / 2 ? slabs * 16 : 0);   // two workgroups per compute unit where it can be
        if (score <= best) { best = score; out.ks = int(ks); out.slabs = int(slabs); out.stages = stages; out.lds = lds; }
    }
    if (best == INT64_MAX) return false;
    // Two slabs on their way instead of one where a workgroup is alone on its compute unit for a long reduction (600 x 990 x 2250 in 60 x 110, 90
    // workgroups x 71 slabs, 29.2 -> 25.3 us; 900 x 1080 x 3150 in 90 x 90, 120 x 50, 34.3 -> 31.8; but 1200 x 900 x 1310 in 60 x 90, 200 x 41, 16.2 -> 17.3, and with a second
    // workgroup, 840 x 2150 x 1368, 602 x 22, 22.1 -> 24.3; tiles of up to 20 atoms and K >= 448 share the reduction instead); the places of a thread's pieces are kept
    // in registers where there is room for them, else worked out again for every slab.
    const int64_t nw = out.wm * out.wn, held = staging(out.ks, 64 * nw);
    const int64_t fit = std::max<int64_t>(1, std::min(kMaxLds / out.lds, (wgs + 255) / 256));       // workgroups on a compute unit
    const int64_t waves = std::max((nw + 3) / 4, std::min<int64_t>(2, (nw * fit + 3) / 4));
    const int64_t rest = held / 4 * 3 + 4 * out.mi * out.ni + 8 * (out.mi + out.ni) + 48;
    out.depth = out.stages == 2 && wgs <= 256 && out.slabs >= 16 && 2 * held + rest <= 512 / waves ? 2 : 1;
    // (2: up to 15 % over, where the compiler fits most of them all the same, is for it to say.  19 such members, two stages, 1.12 to 1.38 times as fast with kept
    // places as without, all 19 within the registers: 1620 x 252 x 1419, 4 x 3 atoms, 68.5 -> 51.4 us; 760 x 594 x 513, 6 x 5 atoms, 30.2 -> 27.0.)
    const int64_t need = out.depth * held + rest, have = 512 / waves;
    out.keep = out.slabs < 2 || 20 * need > 23 * have ? 0 : need > have ? 2 : 1;
    out.min_waves = int(out.keep == 1 ? waves : (nw + 3) / 4);
    return true;
}

// How the few-channels convolution template runs a box: atom, wave grid, atoms per wave, padded kernel row, LDS bytes.
struct Rows { int atom = 0, wm = 0, wn = 0, mi = 0, ni = 0, wkp = 0, persist = 0, stage = 0; int64_t lds = 0, beside = 0; };   // beside: what of lds is the kernel's own array

static bool plan_rows(const opevo_op &op, int64_t bm, int64_t nb2, int64_t bh, int64_t bw, int64_t boxes, int64_t m1, bool linear, Rows &out)
{
    // Boxes of fewer than 4 pixels across re-use too little of a staged row.  Elements are addressed with 31 bits inside the
    // kernel tensor and inside the images of a box.
    if (op.cin >= 16 || op.wk > 16 || op.win < 8 || bw < 4 || bm % 16 != 0 || op.a_elems() >= (int64_t(1) << 31) || op.a_elems() < 8 ||
        nb2 * op.cin * op.hin * op.win >= (int64_t(1) << 31))
        return false;
    const int64_t atom = bm % 32 == 0 ? 32 : 16, q = op.wk <= 8 ? 1 : 2, rps = (atom == 32 ? 2 : 4) / q;   // rps: kernel rows per MFMA step
    const int64_t spc = (op.hk + rps - 1) / rps, steps = op.cin * spc, bn = nb2 * bh * bw;
    const int64_t ph = (bh - 1) * op.stride + op.hk, pitch = ((bw - 1) * op.stride + op.wk + 7) / 8 * 8;
    const int64_t copy = (nb2 * op.cin * ph + spc * rps - op.hk) * pitch + q * 8;
    const int64_t lds = op.stride % 2 ? 2 * ((copy + 127) / 128 * 128 + 64) * 2 : (copy + 7) / 8 * 8 * 2;
    if (lds > kMaxLds) return false;
    const int64_t ma = bm / atom, na = (bn + atom - 1) / atom;
    int64_t best = INT64_MAX;
    for (int64_t wm = 1; wm <= std::min<int64_t>(ma, 8); ++wm)
        for (int64_t wn = 1; ma % wm == 0 && wn <= std::min<int64_t>(na, 8 / wm); ++wn) {
            const int64_t mi = ma / wm, ni = (na + wn - 1) / wn, nw = wm * wn;
            // registers of a lane (256: two waves on every SIMD): the kernel tensor's fragments, and the accumulators beside two sets of
            // the image's fragments or the 16 pieces of the fill
            const int64_t regs = 4 * steps * mi + std::max<int64_t>(mi * ni * (atom == 32 ? 16 : 4) + 8 * ni, 64) + 28;
            if (regs > 256 || steps * mi * ni > 1024) continue;
            // cycles of a box: the MFMAs of the SIMD with the most waves, or the fragment reads of all waves at 128 bytes a
            // cycle; more than four waves leave no room for a second workgroup to load while this one multiplies
            const int64_t mfma = steps * mi * ni * (atom == 32 ? 32 : 16) * ((nw + 3) / 4), reads = nw * steps * ni * 8;
            const int64_t score = std::max(mfma, reads) * (nw > 4 ? 3 : 2) + std::min(mfma, reads);
            if (score < best) { best = score; out.wm = int(wm); out.wn = int(wn); out.mi = int(mi); out.ni = int(ni); }
        }
    if (best == INT64_MAX) return false;
    out.atom = int(atom); out.wkp = int(q * 8); out.lds = lds;
    // The kernel tensor's rows come through the LDS, where the patch will be (1) or, if that is smaller, beside it (2), as long as the compute unit holds
    // as many workgroups with it.  Drawn members 1.03 - 1.85 times as fast as with fragments straight from memory (0), 44 random ones 0.97 - 1.98, 1.16x in the geometric mean.
    const int64_t rows_bytes = (bm * op.K + 128) * 2;
    out.stage = rows_bytes <= lds ? 1 : rows_bytes <= 65536 && (lds + rows_bytes) * std::max<int64_t>(1, 8 / (out.wm * out.wn)) <= kMaxLds ? 2 : 0;
    if (out.stage == 2) { out.beside = rows_bytes; out.lds += rows_bytes; }
    // with four and more boxes for every workgroup the chip holds, that many workgroups take them in turn and fetch the kernel
    // tensor once
    const int64_t resident = 256 * std::max<int64_t>(1, std::min<int64_t>(8 / (out.wm * out.wn), kMaxLds / lds));
    if (!linear && boxes * m1 >= 4 * resident) out.persist = int(std::max<int64_t>(1, resident / m1 / 8) * 8);
    return true;
}

// How the row-strip template runs a box of bm output channels x nb2 images x bh x bw pixels: atom, channels per slab, waves along the
// channels, rows per wave, waves that share a wave tile.
// kw_min: the patch template's division has that many partial sums per output, and so has this one, or more: with fewer the rounding errors of
// the longer chains would be larger (2304 products: 1.8e-7 of the norm in two partial sums, 2.7e-7 in one, 1.6e-7 in three).
struct Strip { int atom = 0, cs = 0, wm = 0, mi = 0, rows = 0, wn = 0, kw = 0, pitch = 0, min_waves = 0; int64_t lds = 0; };

static bool plan_strip(const opevo_op &op, int64_t bm, int64_t nb2, int64_t bh, int64_t bw, int64_t wgs, int64_t kw_min, Strip &out)
{
    // Left to the patch template, by what was measured there: 1 x 1 kernels, which have no rows to re-use, with boxes of part of a row (96 -> 32
    // channels at 56 x 56 9.2 -> 10.0 us) or slabs of 32 channels (96 -> 128 at 27 x 27 6.7 -> 7.1); fewer than two waves on every SIMD (32 -> 64 channels,
    // 5 x 5, boxes of 3 rows of 27 17.2 -> 18.6) or four waves in a workgroup (48 -> 192, 5 x 5, 36 workgroups 10.6 -> 14.8); sharing of
    // a tile with slabs of 16 channels or a single slab (48 -> 192, 3 x 3 5.2 -> 6.6); wave tiles of 32 x 32 atoms that read more than 9
    // fragments for 8 MFMAs (48 -> 128, 3 x 3, two rows a wave 15.4 -> 16.2); more than half the LDS where the grid has a second
    // workgroup for the compute unit (32 -> 192, 5 x 5, 810 workgroups 21.4 -> 23.7).
    if (op.stride != 1 || (op.hk * op.wk == 1 && bw != op.wout)) return false;
    const int64_t taps = op.hk * op.wk, ph = bh + op.hk - 1, pw = bw + op.wk - 1, pitch = (pw + 15) / 16 * 16;
    double best = 1e300;
    for (int64_t atom = 16; atom <= 32; atom += 16)
        for (int64_t cs = atom == 16 ? 32 : 16; cs <= 128; cs *= 2) {
            const int64_t ka = atom == 16 ? 32 : 16, strips = (bw + atom - 1) / atom, units = cs / ka * op.wk, nacc = atom == 16 ? 4 : 16;
            if (bm % atom != 0 || op.cin % cs != 0 || 4 * strips * atom > 5 * bw) continue;   // at least four lanes of five have a pixel
            for (int64_t wm = 1; wm <= 8; ++wm)
                for (int64_t rows = 2; rows <= bh; ++rows)
                    for (int64_t kw = kw_min; kw <= 8; ++kw) {
                        if (bm / atom % wm != 0 || bh % rows != 0 || units % kw != 0) continue;
                        const int64_t wn = nb2 * strips * (bh / rows), nw = wm * wn * kw, nt = 64 * nw, mi = bm / atom / wm;
                        if (nw > kMaxThreads / 64 || (nw < 4 && wgs <= 512) || (kw > 1 && (atom == 32 || op.cin == cs))) continue;
                        const int64_t stage = nb2 * ph * pitch * cs + taps * bm * cs, slabs = op.cin / cs;
                        const int64_t lds = std::max<int64_t>((stage + 512) * 2, kw > 1 ? nw * (nacc / 4) * 1024 : 0);
                        // registers of a lane: accumulators, the fill's plan, and two sets of a unit's fragments or the larger part's data
                        const int64_t fill_p = (cs / 8 * (pw / 2 + 1) * ph * nb2 + nt - 1) / nt, fill_a = (bm * cs / 2 + nt - 1) / nt;
                        const int64_t acc = mi * rows * nacc;
                        const int64_t regs = acc + 3 * fill_p + 2 * fill_a + std::max(4 * (2 * op.hk * mi + 6), std::max(8 * fill_p, taps * fill_a)) + 30;
                        const int64_t mfmas = units / kw * op.hk * rows * mi;       // of a wave and slab
                        const int64_t frags = op.hk * mi + rows + op.hk - 1;        // fragments a unit reads
                        if (lds > kMaxLds || acc > kMaxAcc || regs > 512 / ((nw + 3) / 4) || mfmas > 768) continue;
                        if ((atom == 32 && 8 * frags > 9 * op.hk * rows * mi) || (wgs > 256 && 2 * lds > kMaxLds) || (taps == 1 && cs < 64)) continue;
                        int64_t k = 1;                                              // workgroups a compute unit holds
                        while (k < 8 && (k + 1) * lds <= kMaxLds && nw * (k + 1) <= 32 && regs <= 512 / ((nw * (k + 1) + 3) / 4)) ++k;
                        k = std::max<int64_t>(1, std::min(k, (wgs + 255) / 256));
                        if (nw * k < 8) continue;
                        // Cycles of the k workgroups of a compute unit: what they keep busy together (matrix pipes, LDS), or one of them with
                        // its exposed fill; a SIMD with few waves waits for its own latencies.  Of the forms of this sum tried on 133 compiled divisions of
                        // 16 operators, this one's choice was on average 3 % slower than the fastest of each operator.
                        const double mfma = double((nw + 3) / 4) * mfmas * (atom == 16 ? 16 : 32) * slabs;
                        const double reads = double(nw) * (units / kw) * frags * 8 * slabs;
                        const double stores = double(stage) * 2 / 128 * 2 * slabs, final_sum = kw > 1 ? double(acc) * nw * 8 : 0.0;
                        const double own = slabs * (8.0 * fill_p + double(taps) * fill_a) * 6 + acc * 6.0;   // a wave's own loads, packing and stores
                        const double together = std::max(mfma, reads + stores) * k * (1.0 + 1.0 / std::min(nw * k / 4.0, 8.0));
                        const double alone = (mfma + stores + 4.0 * stores / slabs + 1000.0 * slabs + own + final_sum) * (1.0 + 1.0 / std::max(nw / 4.0, 1.0));
                        const double cost = std::max(1.0, wgs / (256.0 * k)) * std::max(together, alone);
                        if (cost >= best) continue;
                        best = cost;
                        out.atom = int(atom); out.cs = int(cs); out.wm = int(wm); out.mi = int(mi); out.rows = int(rows); out.wn = int(wn); out.kw = int(kw);
                        out.pitch = int(pitch); out.min_waves = int(std::min<int64_t>(8, (nw * k + 3) / 4)); out.lds = lds;
                    }
        }
    return best < 1e300;
}

// How the workgroups of a MatMul / BatchMatMul grid are dealt to tiles.  Consecutive workgroups go to the eight XCDs in turn, each with
// an L2 of its own, so that in the launch's natural order (0) an XCD walks every eighth tile: columns that share cache lines, and the tiles of
// one batch, are spread over all eight.  1 / 2: an XCD walks a contiguous eighth of the tiles, columns / rows first.
// The choice compares the bytes per reduction row that the tiles an XCD has under way at a time take from beyond its L2; a
// column panel that is not surrounded by its neighbours also pays for the rest of its cache lines.
// Measured, natural / columns first / rows first (us): 245 x 7650 x 1590 in 7 x 30 257 / 150 / 108; 2496 x 7072 x 6848 in 64 x 32 1040 / 697 / 749; 6680 x 1650 x 400 in
// 40 x 30 74 / 68 / 83; 506 x (128 x 160 x 160) in 128 x 32 28 / 17 / 18; 8192^3 in 256 x 256 890 / 942 / 995; 512 x 4096 x 1024 fp32 in 64 x 64 47 / 51 / 48.
// The order alone (the rest compiled alike): 43 scalar members 1.13x in the geometric mean (0.92 - 1.76), 25 folded scalar ones 1.07x (0.83 - 1.40), 118 register-staged ones
// 1.19x (0.91 - 2.21), 50 on the fp32 and ragged templates 1.16x (0.97 - 1.78); no line was found around the slower ones.
// Operands that an L2 holds gain nothing and pay for the division (1000^3 in 20 x 100 13.6 / 14.2 / 14.1, 6048 x 108 x 75 3.4 / 3.6 / 3.7), nor do
// small batches (52 x (224 x 192 x 64), 12 MB 5.1 / 5.5 / 5.5): from 4 MiB of operands on, or 16 MB of traffic with batches.
static int xcd_walk(const opevo_op &op, int64_t n1, int64_t m1, int64_t b1, int64_t bm, int64_t bn, int64_t binner, int64_t resident, bool matrix)
{
    auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const int64_t e = op.elem_size(), tiles = n1 * m1;
    int64_t W = 32 * std::max<int64_t>(1, std::min<int64_t>(8, resident));      // tiles an XCD has under way
    auto alone = [&](int64_t w) { return w * e + (w * e % 128 == 0 ? 0 : w * e % 64 == 0 ? 64 : 126); };
    const int64_t row = op.trans_a && m1 > 1 ? alone(bm) : bm * e, col = n1 > 1 ? alone(bn) : bn * e;
    // natural order over a window of `tiles_in` tiles: an XCD's distinct columns and rows
    auto natural = [&](int64_t tiles_in) {
        const int64_t r = std::min(m1, up(tiles_in, n1));
        const int64_t c = std::min(n1, up(n1, 8) * std::min<int64_t>(8 / std::gcd<int64_t>(n1, 8), r));
        return double(c * col + r * row);
    };
    if (tiles * b1 < 64) return 0;
    if (b1 > 1) {
        const double mine = std::max(1.0, tiles / 8.0);                  // tiles of a batch that one XCD has
        const double nat = std::min(natural(tiles) / mine, double(col + row)), walk = double(n1 * bn * e + m1 * bm * e) / tiles;
        return nat * double(op.K) * double(tiles) * double(b1 * binner) >= 16e6 && walk < 0.75 * nat ? 1 : 0;
    }
    if ((op.a_elems() + op.b_elems()) * e <= (int64_t(4) << 20)) return 0;
    // Grids that do not fill the chip: an XCD has an eighth of the tiles.  On the matrix templates and with reductions of 2100 bytes and more 41 drawn members 1.10x in
    // the geometric mean (0.98 - 1.57: 2112 x 128 x 4064 in 64 x 64 18.0 -> 13.2 us, 180 x 1056 x 3267 in 60 x 32 17.1 -> 11.2), 26 further ones 0.99 - 1.64x.  The line is on the safe
    // side: short ones can pay for the division (96 x 4224 x 896 4.51 -> 4.68, 4352 x 96 x 480 6.15 -> 6.34), most gain (18 members of 832 - 2000 bytes 0.97 - 1.62x, 1.19x).  40 random ragged members 1.14x (0.96 - 1.86).  39 random scalar members gain less and lose more (1.06x, 0.94 - 1.40).
    if (matrix && op.K * e >= 2100) W = std::min(W, up(tiles, 8));
    const double nat = natural(std::min(tiles, 8 * W));
    const double by_col = double(std::min(n1, W) * bn * e + 128 + up(W, n1) * row), by_row = double(up(W, m1) * bn * e + 128 + std::min(m1, W) * bm * e);
    if (std::min(by_col, by_row) >= 0.75 * nat) return 0;
    return by_col <= by_row ? 1 : 2;
}

// Members that cannot run without the few-channels template, or the one that takes fp32 values apart (a slab with too many staging registers, or
// too long for the LDS, say), stay invalid: which members of a space are valid does not depend on them.
static bool valid_without_extras(const opevo_op &op, int variant, const int32_t *cfg)
{
    Decoded d;
    return decode(op, variant, cfg, d, false) == OPEVO_OK && d.plan.status == OPEVO_OK;
}

static void invalid(opevo_plan &p, const char *fmt, long a = 0, long b = 0)
{
    p.status = OPEVO_E_INVALID;
    snprintf(p.reason, sizeof p.reason, fmt, a, b);
}

int decode(const opevo_op &op, int variant, const int32_t *cfg, Decoded &out, bool extras)
{
    std::vector<opevo_param_desc> descs;
    if (int rc = op_param_descs(op, variant, descs)) return rc;
    // legality: every factor tuple multiplies back to its axis, flags in range
    {
        int off = 0;
        for (const auto &d : descs) {
            if (d.type == OPEVO_FACTOR) {
                int64_t prod = 1;
                for (int j = 0; j < d.nu; ++j) {
                    if (cfg[off + j] < 1) return fail(OPEVO_E_ILLEGAL, "factor %d of %s is < 1", j, d.name);
                    prod *= cfg[off + j];
                    if (prod > d.C) break;
                }
                if (prod != d.C)
                    return fail(OPEVO_E_ILLEGAL, "factors of %s do not multiply to %lld", d.name, (long long)d.C);
                off += d.nu;
            } else if (d.type == OPEVO_PERMUTATION) {
                unsigned seen = 0;
                for (int j = 0; j < d.n_values; ++j) {
                    if (cfg[off + j] < 0 || cfg[off + j] >= d.n_values || (seen >> cfg[off + j] & 1u))
                        return fail(OPEVO_E_ILLEGAL, "%s is not a permutation of 0..%d", d.name, d.n_values - 1);
                    seen |= 1u << cfg[off + j];
                }
                off += d.n_values;
            } else {
                if (cfg[off] < 0 || cfg[off] >= d.n_values)
                    return fail(OPEVO_E_ILLEGAL, "%s out of range", d.name);
                off += 1;
            }
        }
    }

    opevo_plan &p = out.plan;
    std::memset(&p, 0, sizeof p);
    p.status = OPEVO_OK;
    std::ostringstream D;

    // ---- common GEMM-view quantities filled by each variant
    int64_t m1 = 1, n1 = 1, b1 = 1, binner = 1;
    int64_t BM = 1, BN = 1, BK = 1, ksteps = 1, WM = 1, WN = 1, TM = 1, TN = 1, FM = 1, FN = 1;
    int flagv = 0;
    int64_t nb2 = 1, BH = 1, BW = 1, h1 = 1, w1 = 1;
    bool four_level = (variant == OPEVO_TILE4 || variant == OPEVO_TILE4X || variant == OPEVO_TILE4P || variant == OPEVO_TILE4K ||
                       variant == OPEVO_TILE4C || variant == OPEVO_TILE4T || variant == OPEVO_TILE4A || variant == OPEVO_TILE4L);
    int atom16 = 0;                        // MatMul, TILE4A: 1 = 16x16x32 atoms on direct-to-LDS members
    int bpack = 0;                         // MatMul, TILE4T: 1 = second operand transposed to [N][K] by a pre-pass
    int layout = 0;                        // Conv2d, TILE4C: 1 = channels-last operands (pre-pass)
    int64_t subm = 1, subn = 1;            // sub-tiles a workgroup computes one after another (folded members)
    int64_t ksplit = 1;
    int64_t box[6] = {1, 1, 1, 1, 1, 1};   // C_in, H_k, W_k as (boxes, box extent) pairs
    bool tap_box = false;
    int64_t kunroll = 0;                   // 0: the template's default
    int64_t patch_cs = 0;                  // Conv2d, TILE4L, layout 2: channels per slab of the LDS-resident patch (0: not on that template)
    int patch_atom = 0, patch_stages = 1, patch_kw = 1;
    int64_t patch_row = 0, patch_image = 0;   // its row pitch and image pitch in pixels
    Strip strip;                              // strip.rows > 0: such a member on the row-strip template instead
    int tile4_width = 0;   // slots of the four-level part, after which the launch-order parameters follow

    if (!four_level) {
        m1 = cfg[0]; BM = cfg[1]; n1 = cfg[2]; BN = cfg[3]; ksteps = cfg[4]; BK = cfg[5];
        flagv = 1;
    } else if (op.kind == OPEVO_MATMUL || op.kind == OPEVO_BMM) {
        const int32_t *c = cfg;
        if (op.kind == OPEVO_BMM) { b1 = c[0]; binner = c[1]; c += 2; }
        m1 = c[0]; WM = c[1]; TM = int64_t(c[2]) * c[3]; FM = c[3];
        n1 = c[4]; WN = c[5]; TN = int64_t(c[6]) * c[7]; FN = c[7];
        if (variant == OPEVO_TILE4K) { ksplit = c[8]; b1 = ksplit; ksteps = c[9]; BK = c[10]; flagv = c[11]; }
        else { ksteps = c[8]; BK = c[9]; flagv = c[10]; }
        if (variant == OPEVO_TILE4T) bpack = c[11];
        if (variant == OPEVO_TILE4A) atom16 = c[11];
        BM = WM * TM; BN = WN * TN;
        tile4_width = int(c - cfg) + (variant == OPEVO_TILE4K || variant == OPEVO_TILE4T || variant == OPEVO_TILE4A ? 12 : 11);
    } else {   // conv: B(2) Cout(4) H(4) W(4) R(2) flag
        const int32_t *c = cfg;
        const int64_t nb1 = c[0]; nb2 = c[1];
        m1 = c[2]; WM = c[3]; TM = int64_t(c[4]) * c[5]; FM = c[5];
        const int32_t *h = c + 6, *w = c + 10;
        h1 = h[0]; w1 = w[0];
        BH = int64_t(h[1]) * h[2] * h[3]; BW = int64_t(w[1]) * w[2] * w[3];
        WN = int64_t(h[1]) * w[1];
        TN = nb2 * h[2] * h[3] * w[2] * w[3];
        FN = nb2 * h[3] * w[3];
        n1 = nb1 * h1 * w1;
        if (variant == OPEVO_TILE4P) {
            for (int j = 0; j < 6; ++j) box[j] = c[14 + j];
            ksteps = box[0] * box[2] * box[4];
            BK = box[1] * box[3] * box[5];
            flagv = c[20];
            kunroll = int64_t(kUnrollSteps[c[21]]);
            // a box that spans whole kernel rows (and whole kernel planes if it holds several
            // channels) is a contiguous run of the flattened reduction axis: the plain walk
            const bool contiguous = (box[5] == op.wk || (box[3] == 1 && box[1] == 1)) && (box[3] == op.hk || box[1] == 1);
            tap_box = !contiguous;
            tile4_width = 22;
        } else if (variant == OPEVO_TILE4C) {
            ksplit = c[14]; b1 = ksplit; ksteps = c[15]; BK = c[16]; flagv = c[17]; layout = c[18];
            tile4_width = 19;
        } else if (variant == OPEVO_TILE4L) {
            const int64_t taps = op.hk * op.wk;
            flagv = c[16];
            tile4_width = 19;
            if (c[17] == 1) { layout = 1; ksteps = taps * c[14]; BK = c[15]; }   // channels-last walk (r, s, ci): a slab is c[15] channels of one tap
            else { ksteps = c[14]; BK = c[15] * taps; }                          // walk (ci, r, s): a slab is c[15] channels with all their taps
            // layout 2: the LDS-resident patch, for members it can hold (the others run as with layout 0).
            // 32x32x16 atoms need slabs of whole 16 channels, 16x16x32 atoms of 32; the wave's pixel side is
            // rounded up to whole atoms while that at most doubles the work; the atom that wastes less is taken.
            // kwaves: that many waves share every wave tile and split the MFMA steps of a slab (taps x channel groups).
            // A member that asks for what the template has not is folded rather than sent away (same workgroup tile,
            // another division of it among the waves): slabs of fewer than 16 channels are merged, slabs too long for the
            // LDS halved; wave tiles of fewer than 16 output channels are merged along Cout; with more than 16 waves kwaves
            // is halved, then the waves along the pixels are merged a prime at a time (their tiles grow).
            if (c[17] == 2 && op.dtype != OPEVO_F32 && op.win >= 2 && op.b_elems() < (int64_t(1) << 30) && op.a_elems() < (int64_t(1) << 30)) {
                auto up = [](int64_t v, int64_t a) { return (v + a - 1) / a * a; };
                auto prime = [](int64_t n) { for (int64_t q = 2; q * q <= n; ++q) if (n % q == 0) return q; return n; };
                int64_t cs = c[15], tm = TM, wm = WM;
                while (cs % 16 != 0 && cs < op.cin) cs *= prime(op.cin / cs);
                // ... and slabs too long for the LDS (the kernel tensor's part holds all taps of a slab) are halved while they
                // stay whole 16 channels
                {
                    int64_t prow0 = 0, pimage0 = 0;
                    patch_pitches(op, BH, BW, false, prow0, pimage0);
                    auto stage_bytes = [&](int64_t v) { return (nb2 * pimage0 * (v + 8) + taps * WM * TM * v + 64) * 2; };
                    while (cs % 32 == 0 && stage_bytes(cs) * ((flagv && op.cin / cs > 1) ? 2 : 1) > kMaxLds) cs /= 2;
                }
                const int64_t slabs = op.cin / cs;
                const int64_t ph = (BH - 1) * op.stride + op.hk, pw = (BW - 1) * op.stride + op.wk;
                const int st = (flagv && slabs > 1) ? 2 : 1;
                // the padded pitches if the LDS has room for them, else the plain ones
                int64_t prow = 0, pimage = 0, lds_p = 0;
                for (int padded = 1; padded >= 0; --padded) {
                    patch_pitches(op, BH, BW, padded == 1, prow, pimage);
                    lds_p = st * (nb2 * pimage * (cs + 8) + taps * wm * tm * cs + 64) * 2;   // patch (padded pixels), kernel tensor's part, dump words
                    if (lds_p <= kMaxLds) break;
                }
                // the waves along Cout are merged, a prime at a time, until an atom fits the wave tile
                for (; !patch_cs; ) {
                    for (int64_t kw = int64_t(kReductionWaves[c[18]]); kw >= 1 && !patch_cs && tm % 16 == 0; kw /= 2) {
                        int64_t wn = WN, tn = TN;
                        while (wm * wn * kw > kMaxThreads / 64 && wn > 1) { const int64_t q = prime(wn); wn /= q; tn *= q; }
                        if (64 * wm * wn * kw > kMaxThreads) continue;
                        auto fits = [&](int64_t at) {
                            return tm % at == 0 && cs % (at == 32 ? 16 : 32) == 0 && up(tn, at) <= 2 * tn && tm * up(tn, at) <= 64 * kMaxAcc;
                        };
                        const int at = fits(32) && (!fits(16) || up(tn, 32) == up(tn, 16)) ? 32 : fits(16) ? 16 : 0;
                        if (!at) continue;
                        // the fill: per thread, tasks of two channels x two pixels (images one pixel wide, which the template would fill pixel by pixel, stay with layout 0) and of two channels x all taps (kernel tensor)
                        // (w: the waves that share a tile)
                        auto room = [&](int64_t w) {
                            const int64_t nw = wm * wn * w, nt = 64 * nw;
                            if (w > taps * (cs / (at == 32 ? 16 : 32))) return false;   // more waves than steps
                            const int64_t fill_p = (cs / 2 * (op.win >= 2 ? pw / 2 + 1 : pw) * ph * nb2 + nt - 1) / nt, fill_a = (wm * tm * cs / 2 + nt - 1) / nt;
                            // Registers: a lane has 512 / (waves per SIMD).  Counted: the accumulators, two sets of fragments (4 per
                            // atom row and column; three sets for small wave tiles), the fill (3 + 2 per image task, 2 + taps per
                            // kernel-tensor task: plan + data in flight), 24 for addresses, and where waves share a tile 40 + three
                            // quarters of the accumulators again (the final sum moves them through ordinary registers).  An eighth
                            // over is let through: the compiler fits such members.  Calibrated on compiled members: of 150 random
                            // eligible ones the rule lets no spilling member through and turns away 3 that would have fitted; a
                            // member that spills all the same is refused when its kernel is loaded.
                            const int64_t fill = 5 * fill_p + (2 + taps) * fill_a;
                            const int64_t accs = tm * up(tn, at) / 64;
                            const int64_t frags = tm / at + up(tn, at) / at;
                            const int64_t need = accs + (frags <= 3 ? 12 : 8) * frags + 24 + fill + (w > 1 ? 40 + accs * 3 / 4 : 0);
                            const int64_t have = 512 / ((nw + 3) / 4);
                            // adding the partial sums of kw waves needs room for one atom of every wave
                            const int64_t lds_r = w > 1 ? nw * (at == 32 ? 4 : 1) * 1024 : 0;
                            return lds_p <= kMaxLds && lds_r <= kMaxLds && need <= have + have / 8;
                        };
                        if (room(kw)) {
                            patch_cs = cs; patch_atom = at; patch_stages = st; patch_row = prow; patch_image = pimage; patch_kw = int(kw);
                            // Workgroups of one or two waves that do not fill the chip get waves that share a tile although the member
                            // asks for none: nothing else hides a fragment read there, and the fill is shared as well.  Measured, bf16,
                            // 80 members of up to 512 workgroups, 1.00 to 2.1 times as fast: 12 x 256 x 13 x 13 * 96 x 256 x 5 x 5 as 36
                            // workgroups of one wave 68.2 -> 31.9 us, 6 x 96 x 13 x 13 * 128 x 96 x 5 x 5 as 12 of two waves 28.1 -> 20.1.
                            // Past one workgroup per compute unit: one wave as 475: 11.4 -> 10.7 with two, 10.6 with four; as 550: 20.5 ->
                            // 20.5 and 26.2; two waves as 453 (32 accumulators a lane) 24.2 -> 22.8, but as 472 (96: a second workgroup no
                            // longer finds registers) 18.4 -> 22.2.  Workgroups of three and more waves gain nothing or lose.
                            if (extras && c[18] == 0 && wm * wn <= 2) {
                                const int64_t wgs = n1 * m1;
                                const bool fits_twice = wm * wn == 1 || tm * up(tn, at) <= 64 * 64;
                                for (int64_t more = wgs > 512 || (wgs > 256 && !fits_twice) ? 1 : wm * wn == 1 && wgs <= 256 ? 4 : 2; more > 1 && patch_kw == 1; more /= 2)
                                    if (room(more)) { patch_kw = int(more); out.extra_waves = true; }
                            }
                            // the member as the template runs it
                            WM = wm; TM = tm; WN = wn; TN = tn; FM = std::gcd(FM, TM); FN = std::gcd(FN, TN);
                            ksteps = slabs; BK = cs * taps;
                        }
                    }
                    if (wm == 1) break;
                    const int64_t q = prime(wm); wm /= q; tm *= q;
                }
                // Members that have to be divided anew anyway, because they ask for more waves than a workgroup holds, and members that ask for no
                // pipelining and no sharing and deal their pixels to several waves, go to the row-strip template where it has a division
                // (the others run the loop and the division that they ask for).  144 drawn members and 60 folded ones of 8 operators, old
                // template against new: 1.20 - 1.26x in the geometric mean, 0.94 - 2.5x; what was below 0.94 is excluded by the conditions in plan_strip.
                // Members that ask for pipelining go there too on more workgroups than compute units: the second stage costs them the other workgroups that would
                // hide a slab's latency.  144 drawn and random members with three pixel waves and more 0.94 - 2.7x, 1.3x in the geometric mean (53 x 256 x 27 x 27 *
                // 64 x 256 x 3 x 3 31.2 -> 26.5 us, 163 x 256 x 14 x 14 * 256 x 256 x 3 x 3 74.4 -> 53.3; the slowest 11 x 32 x 56 x 56 * 128 x 32 x 3 x 3 10.9 -> 11.5).  Two pixel waves
                // (11 members 1.4 - 2.4x as fast there) and grids of up to 256 workgroups (17 members 1.04 - 1.30x) were too few to draw a line by: they stay.
                const int64_t asked_n = int64_t(h[1]) * w[1], asked = c[3] * asked_n * int64_t(kReductionWaves[c[18]]);
                if (extras && patch_cs && (asked > kMaxThreads / 64 || (c[18] == 0 && (flagv == 0 ? asked_n >= 2 : asked_n >= 3 && n1 * m1 > 256))) &&
                    plan_strip(op, WM * TM, nb2, BH, BW, n1 * m1, patch_kw, strip)) {
                    out.extra_waves = true;
                    patch_cs = strip.cs; patch_atom = strip.atom; patch_stages = 1; patch_kw = strip.kw;
                    WM = strip.wm; TM = strip.mi * strip.atom; FM = std::gcd(FM, TM);
                    WN = strip.wn; TN = strip.rows * strip.atom; FN = 1;
                    ksteps = op.cin / strip.cs; BK = strip.cs * taps;
                }
            }
        } else {
            ksteps = c[14]; BK = c[15]; flagv = c[16];
            tile4_width = 17;
        }
        BM = WM * TM; BN = strip.rows ? nb2 * BH * BW : WN * TN;
    }
    // ---- members that ask for more than a workgroup has are folded into serial work instead of scoring 0
    // (the search then sees a slow member with its own place in the landscape, not a hole; Sec. 4.2 keeps
    // zero fitness for what cannot run at all):
    //  * a per-wave tile that needs more than 256 accumulators per lane (or, for a member with more than
    //    16 waves, more than its occupancy leaves) is cut along its longer side (a prime at a time) into
    //    sub-tiles, each of which becomes the tile of a wave of its own;
    //  * a reduction slab too long for the LDS is halved (twice as many steps) while it stays a
    //    multiple of 32;
    //  * more than 16 waves (below): the workgroup runs the largest divisor of their number that fits,
    //    and every real wave takes the tiles of several waves one after another, each with the whole K loop.
    if (four_level && !patch_cs) {
        auto smallest_prime = [](int64_t n) { for (int64_t q = 2; q * q <= n; ++q) if (n % q == 0) return q; return n; };
        // The registers a lane may use depend on how many waves share a SIMD (512 for one, 256 for two,
        // 128 for four): a member that is folded anyway gets wave tiles that leave room for fragments
        // and staging next to the accumulators at the occupancy it will run at.
        auto real_waves = [&](int64_t v) { for (int64_t dv = kMaxThreads / 64; dv > 1; --dv) if (v % dv == 0) return dv; return int64_t(1); };
        auto acc_cap = [&]() {
            const int64_t per_simd = (real_waves(WM * WN) + 3) / 4;
            return std::min<int64_t>(kMaxAcc, 512 / per_simd / 2 - 8);   // half the registers: the other half holds two slabs in flight and the fragments
        };
        const bool refold = TM * TN > 64 * kMaxAcc || WM * WN > kMaxThreads / 64;
        while (refold && TM * TN > 64 * acc_cap() && TM * TN > 1) {
            const bool cut_m = (TM >= TN && TM > 1) || TN == 1;
            int64_t &T = cut_m ? TM : TN, &W = cut_m ? WM : WN, &F = cut_m ? FM : FN;
            const int64_t q = smallest_prime(T);
            T /= q; W *= q;
            F = std::gcd(F, T);
        }
        //  * a workgroup tile too large for the LDS even with the shortest slab (or, on the scalar template,
        //    for 1024 threads with 256 outputs each) is cut, a prime at a time along its longer side, into
        //    sub-tiles that the workgroup computes one after another (SUBM x SUBN of them).
        const int elem = op.dtype == OPEVO_F32 ? 4 : 2;
        const int stages = (flagv && ksteps > 1) ? 2 : 1;
        auto lds_need = [&]() { return (BM + BN) * std::max<int64_t>((BK + kPad) * elem * stages, BK * 4); };
        const int64_t lds_cap = kMaxLds - 16;   // room for the deadline flag word of folded members
        // (TILE4L's gather members walk (ci, r, s) in slabs of whole channels with all their taps, rarely a multiple of 64:
        // there a slab too long is divided by its smallest prime factor; the gather pads any slab to the MFMA step)
        if (variant == OPEVO_TILE4L && layout != 1)
            while (lds_need() > lds_cap && BK > 32) { const int64_t q = smallest_prime(BK); BK /= q; ksteps *= q; }
        while (lds_need() > lds_cap && BK % 64 == 0 && !tap_box) { BK /= 2; ksteps *= 2; }
        // (the scalar template: 1024 threads have 128 registers per lane each; 16 outputs per thread fit with its unrolled loop)
        const int64_t out_cap = BM * BN > int64_t(kMaxThreads) * kMaxAcc ? int64_t(kMaxThreads) * 16 : INT64_MAX;
        while (lds_need() > lds_cap || BM * BN > out_cap) {
            // a convolution's column block is a box of pixels: only its channel side is cut
            const bool cut_m = op.kind == OPEVO_CONV2D || BM >= BN;
            int64_t &W = cut_m ? WM : WN, &T = cut_m ? TM : TN, &F = cut_m ? FM : FN, &S = cut_m ? subm : subn;
            if (W * T == 1) break;
            if (W > 1) { const int64_t q = smallest_prime(W); W /= q; S *= q; }
            else { const int64_t q = smallest_prime(T); T /= q; S *= q; F = std::gcd(F, T); }
            BM = WM * TM; BN = WN * TN;
        }
    }
    // extended variant: launch order and group width
    const bool linear = (variant == OPEVO_TILE4X);
    int order[3] = {0, 1, 2};
    int64_t group = 1;
    if (linear) {
        const int n_axes = op.kind == OPEVO_BMM ? 3 : 2;
        for (int j = 0; j < n_axes; ++j) order[j] = cfg[tile4_width + j];
        group = int64_t(kGroupValues[cfg[tile4_width + n_axes]]);
    }

    // ---- template choice
    int path = 0;   // scalar
    int64_t BKP = BK;   // width of a K slab as the MFMA template stages and multiplies it
    int64_t TMacc = TM, TNacc = TN;   // wave tile in whole atoms (accumulator registers)
    bool ragged = false;
    // Channels-last operands (TILE4C, layout = 1) need 8-value pieces that never straddle a tap (Cin and
    // the LDS tile multiples of 8) and byte offsets into the image that fit 32 bits; they exist on the
    // MFMA templates only.  Elsewhere the choice is inert and the member runs as with layout = 0.
    const bool nhwc_ok = layout == 1 && op.kind == OPEVO_CONV2D && op.dtype != OPEVO_F32 && op.cin % 8 == 0 &&
                         BK % 8 == 0 && op.b_elems() * 2 + 256 < (int64_t(1) << 32) &&
                         op.hin + 2 * op.pad + op.hk < 32768 && op.win + 2 * op.pad + op.wk < 32768;   // coordinates in 15 bits
    int nstage_dlds = 0;
    bool dlds_atom16 = false;
    int64_t bnr = BN;   // rows of the second operand's stage part on the direct-to-LDS template when it is K-contiguous
    int64_t anr = BM;   // rows of the first operand's stage part there
    // Direct global->LDS streaming (path 3) of a pipelined member whose slabs split into whole 1 KiB wave
    // loads: `rows_b` rows of BK K-contiguous elements for the second operand (0: it is stored [K][N]).
    auto dlds_stages = [&](int64_t rows_a, int64_t rows_b, bool a_km_rows, bool atoms16 = false) -> int {
        const int64_t nw = WM * WN;
        if (subm * subn > 1) return 0;   // folded members stay on the register-staged template
        if (64 * nw > kMaxThreads || !(BK == 32 || BK == 64 || BK == 128)) return 0;
        const int64_t a_bytes = rows_a * BK * 2, b_bytes = (rows_b ? rows_b : BN) * BK * 2;
        if (a_bytes % (1024 * nw) != 0 || b_bytes % (1024 * nw) != 0) return 0;
        if (!rows_b && !(BN % 128 == 0 || BN == 64 || BN == 32)) return 0;
        if (a_km_rows && !(BM % 128 == 0 || BM == 64 || BM == 32)) return 0;   // A rows are M-contiguous then
        const int64_t per = (a_bytes + b_bytes) / (1024 * nw);
        int st_found = 0;
        for (int st = 4; st >= 2; --st)
            if (st * (a_bytes + b_bytes) <= kMaxLds && (st - 2) * per <= 63) { st_found = st; break; }
        if (!st_found) return 0;
        // The template keeps accumulators and fragments in register arrays and relies on its K
        // loop body (one pass over the ring) unrolling completely.  Instructions in that body:
        // per stage and MFMA step the MFMAs and fragment reads, per stage the loads.  Bodies
        // past this size were seen not to unroll (code objects of 0.5-1.5 MB instead of 20 KB);
        // such members use the register-staged template instead.
        const int64_t at = atoms16 ? 16 : 32;
        const int64_t mi = TM / at, ni = (TN + at - 1) / at, kk = BK / (atoms16 ? 32 : 16);
        const int64_t body = st_found * (kk * (mi * ni + (op.trans_a ? 2 : 1) * mi + (rows_b ? 1 : 2) * ni) + per);
        // 16x16x32 atoms: twice the MFMAs for the same tile; such bodies (up to 128 x 128 wave tiles on slabs of 32)
        // were checked to unroll (code objects of about 30 KiB)
        return body > (atoms16 ? kMaxDldsBody16 : kMaxDldsBody) ? 0 : st_found;
    };
    if (four_level && op.dtype != OPEVO_F32) {
        if (op.kind == OPEVO_CONV2D) {
            // The convolution's reduction axis Cin*Hk*Wk rarely has a factor 16 (3*11*11 = 363): a slab
            // of BK taps is staged zero-padded to the next multiple of the MFMA K step, and its
            // operands are gathered element by element, so no alignment is asked of it.
            // Likewise a wave tile that is no multiple of 16 is rounded up to whole 16x16 atoms as long
            // as that at most doubles the work (pixel tiles come from factors of 55, 27, ...).
            const int64_t TMp = (TM + 15) / 16 * 16, TNp = (TN + 15) / 16 * 16;
            if (TM % 32 == 0 && TN % 32 == 0) { path = 1; BKP = (BK + 15) / 16 * 16; }
            else if (TMp * TNp <= 2 * TM * TN) { path = 2; BKP = (BK + 31) / 32 * 32; ragged = (TMp != TM || TNp != TN); TMacc = TMp; TNacc = TNp; }
            // channels-last, pipelined, wave tiles of whole 32-row atoms whose pixel side rounds up to 32
            // without doubling the work: the direct-to-LDS template with a K-contiguous second operand
            const int64_t TN32 = (TN + 31) / 32 * 32;
            if (nhwc_ok && flagv == 1 && TM % 32 == 0 && TN32 <= 2 * TN && TM * TN32 / 64 <= kMaxAcc) {
                const int64_t nw = WM * WN;
                // rows staged: every pixel of the box and every row a wave's last atom reads, rounded up
                // until the part splits into whole 1 KiB loads per wave
                int64_t rows = std::max(BN, (WN - 1) * TN + TN32), rows_a = BM;
                if (BK == 32 || BK == 64 || BK == 128) {
                    const int64_t unit = 1024 * nw / std::gcd(int64_t(1024) * nw, BK * 2);
                    rows = (rows + unit - 1) / unit * unit;
                    rows_a = (rows_a + unit - 1) / unit * unit;
                    if (rows * BK * 2 / (1024 * nw) <= 16 && rows_a * BK * 2 / (1024 * nw) <= 16)
                        nstage_dlds = dlds_stages(rows_a, rows, false);
                }
                if (nstage_dlds) { path = 3; bnr = rows; anr = rows_a; BKP = BK; ragged = false; TMacc = TM; TNacc = TN32; }
            }
        } else {
            const bool align_ok = (op.K % 8 == 0) && (op.N % 8 == 0);
            if (align_ok && TM % 32 == 0 && TN % 32 == 0 && BK % 16 == 0) path = 1;
            else if (align_ok && TM % 16 == 0 && TN % 16 == 0 && BK % 32 == 0) path = 2;
        }
    }
    // fp32 inputs: 32x32x2 fp32 atoms (MatMul / BMM), both operands in 16-byte pieces along their
    // contiguous axis, K slabs in groups of 8
    if (four_level && op.dtype == OPEVO_F32 && op.kind != OPEVO_CONV2D && TM % 32 == 0 && TN % 32 == 0 &&
        BK % 8 == 0 && op.N % 4 == 0 && (op.trans_a ? op.M % 4 == 0 : op.K % 4 == 0))
        path = 4;
    // fp32 Conv2d: operands gathered value by value, so any slab length (staged padded to 8) and any
    // wave tile whose round-up to whole 32x32 atoms at most doubles the work
    if (four_level && op.dtype == OPEVO_F32 && op.kind == OPEVO_CONV2D) {
        const int64_t TMp = (TM + 31) / 32 * 32, TNp = (TN + 31) / 32 * 32;
        if (TMp * TNp <= 2 * TM * TN && op.b_elems() < (int64_t(1) << 31)) {
            path = 4; BKP = (BK + 7) / 8 * 8; TMacc = TMp; TNacc = TNp;
        }
    }
    if (patch_cs) { path = 5; BKP = BK; ragged = false; TMacc = TM; TNacc = (TN + patch_atom - 1) / patch_atom * patch_atom; }
    const bool stage_lds = path == 4 || !(op.kind == OPEVO_BMM && four_level && flagv == 0 && path != 0);
    // Direct global->LDS streaming (path 3) for pipelined MatMul / BMM members of 32x32 atoms whose
    // slabs split into whole 1 KiB wave loads and whose row lengths suit the chunk permutation.  With
    // bpack = 1 (TILE4T) the second operand is read from the [N][K] copy a pre-pass makes.
    const bool b_packed = bpack == 1 && op.kind == OPEVO_MATMUL && !op.trans_a;
    if (path == 1 && flagv == 1 && stage_lds && op.kind != OPEVO_CONV2D) {
        nstage_dlds = dlds_stages(BM, b_packed ? BN : 0, op.trans_a);
        if (nstage_dlds) path = 3;
        // TILE4A, atom = 1: the same member on 16x16x32 atoms (MatMul with row-major operands; a member whose body
        // would grow too long keeps the 32x32x16 atoms)
        if (nstage_dlds && atom16 == 1 && op.kind == OPEVO_MATMUL && !op.trans_a && !b_packed && BK % 32 == 0 &&
            dlds_stages(BM, 0, false, true) == nstage_dlds && (BK % 64 == 0 || nstage_dlds % 2 == 0))   // one K step per slab: an even ring
            dlds_atom16 = true;
    }
    // MatMul / BMM operators with an extent that is no multiple of 16 have no member on the templates above (or only the few
    // whose tiles skip that axis): their members run on the ragged MFMA template instead of the scalar one.  It takes the
    // workgroup tile as it is, rounds it up to whole 16x16 atoms and deals those to waves by itself.  Measured on 1000^3
    // against the scalar template, one-wave members: tiles of 20 x 100 (atoms of 1.8 times the tile, dealt to four waves 2.05) 15.6 against 1124 us
    // (that tile's best scalar member, 20 waves, 168), 10 x 20 (2.6) 39 against 519, 8 x 8 (4) 79 against 310, 4 x 8 and 8 x 4 (8 times)
    // 144 and 171 against 356 and 381: by about 16 times nothing is left, so the line lies at 8.
    Ragged rg;
    int rg_kw = 0;
    if (four_level && path == 0 && op.dtype != OPEVO_F32 && op.kind != OPEVO_CONV2D && subm * subn == 1 &&
        (op.M % 16 != 0 || op.N % 16 != 0 || op.K % 16 != 0) &&
        plan_ragged(op, BM, BN, BK, op.K / ksplit, n1 * m1 * b1, flagv != 0 || op.kind == OPEVO_BMM, rg)) {
        path = 6;
        WM = rg.wm; WN = rg.wn; TM = rg.mi * 16; TN = rg.ni * 16;
        TMacc = TM; TNacc = TN; BK = rg.ks; ksteps = rg.slabs;
        // Waves that share the reduction, each with the whole tile as its wave tile and a part of the LDS of its own, where no more than one workgroup falls on a compute unit:
        // eight, as far as the LDS goes.  60 drawn and random members of K >= 448 and up to 20 atoms against the slab walk: 0.93 - 2.9x, 1.6x in the geometric mean, 205 further random ones 0.83 - 4.8x, 1.6x, six below 0.98 (480 x 360 x 4893,
        // 90 workgroups, 29.8 -> 21.1 us; 40 x 100 x 2517, 8, 19.8 -> 7.5); below, 56 x 56 at K = 324 4.3 -> 4.6, 32 x 44 at 360 3.2 -> 3.4; with 500 workgroups of 20 x 100
        // at K = 1000 13.2 -> 13.4, with 860 of 50 x 32 32.0 -> 39.6.
        // Two waves on fuller grids where an operand's pieces begin at odd elements, which this loop shifts into place: 190 random members of up to 1024 workgroups and 12 atoms 0.80 -
        // 3.5x, 1.34x in the geometric mean, 18 below 0.98 with no line around them (80 x 3625 x 888 in 40 x 25 8.1 -> 10.2; 100 x 5439 x 1056 in 50 x 21 20.4 -> 11.1; 1078 workgroups 39.9 -> 41.6, 1125 23.9 -> 18.9, 1575 25.8 -> 26.0).
        const int64_t ma = (BM + 15) / 16, na = (BN + 15) / 16, wgs = n1 * m1 * b1;
        const bool odd = op.N % 2 != 0 || (BN % 2 != 0 && n1 > 1) || (op.trans_a && (op.M % 2 != 0 || (BM % 2 != 0 && m1 > 1)));
        auto odd16 = [](int64_t n) { return ((n + 15) / 16 | 1) * 16; };
        const int64_t a_part = op.trans_a ? 32 * odd16(ma * 16) + 192 : ma * 16 * 40, b_part = 32 * odd16(na * 16) + 192;
        const int64_t per = std::max(2 * (a_part + b_part), ma * 16 * (na * 16 + 4) * 4);           // bytes of LDS a wave's operands, or its sums, take
        int64_t kw = 0;
        if (extras && ksplit == 1 && op.K >= 448) kw = wgs <= 256 && ma * na <= 20 ? std::min<int64_t>(8, kMaxLds / per) : odd && op.K >= 500 && wgs <= 1024 && ma * na <= 12 ? 2 : 0;
        if (kw == 2 || kw >= 4) {
            // (256 registers a lane whatever the number of waves: 13 members of two waves 1.00 - 1.04 times as fast as with 512)
            rg_kw = int(kw); rg.lds = kw * per; rg.min_waves = 2;
            out.extra_waves = true;
            WM = 1; WN = kw; TM = ma * 16; TN = na * 16; TMacc = TM; TNacc = TN;
        }
    }
    // Conv2d with fewer than 16 input channels (no slab of whole channels for the patch template): image rows in LDS, taps of a
    // kernel row as the reduction's groups of 8
    Rows rows;
    if (extras && four_level && op.dtype != OPEVO_F32 && op.kind == OPEVO_CONV2D && (path == 0 || path == 1 || path == 2) && !nhwc_ok && subm * subn == 1 &&
        ksplit == 1 && plan_rows(op, BM, nb2, BH, BW, n1, m1, linear, rows) && valid_without_extras(op, variant, cfg)) {
        path = 7;
        WM = rows.wm; WN = rows.wn; TM = rows.mi * rows.atom; TN = rows.ni * rows.atom;
        TMacc = TM; TNacc = TN; BK = op.K; BKP = op.K; ksteps = 1; ragged = false; tap_box = false;
    }
    // Direct-to-LDS MatMul / BMM members of one or two waves (or four on short slabs) whose grid leaves every compute unit
    // at most one workgroup: two groups of waves share the reduction.  A slab of one wave is a chain of latencies of some
    // 0.15 us (64 x 64 x 8192 in 32 x 32 tiles: 22.2 -> 11.2 us; 96 x 160 x 512, 8 steps of 64: 3.40 -> 2.84; 480 x 480 x 1024: 4.81 -> 3.94); with more
    // bytes per slab it is what a compute unit can load (12 KB, 2 waves: 80 workgroups x 32 steps 6.69 -> 5.50 us, x 8 steps 3.35 ->
    // 3.61, 225 workgroups x 32 steps 8.65 -> 9.14; 8 KB, 4 waves: 64 workgroups x 32 steps 4.78 -> 4.48, 256 workgroups 5.56 -> 5.58; 16 KB, 4
    // waves: always slower).  Four groups were nowhere better than two by more than the noise, and slower on most shapes.
    // All of that was measured with wave tiles of one or two 32 x 32 atoms, and the split stays with those: larger ones have MFMAs to cover
    // their latencies with.  It also stays with reductions of more than 256 (96 x 160 x 256 2.68 -> 2.44 us, 480 x 480 x 256 2.82 -> 2.69):
    // a search over the members of 256^3, where one wave often has 4 to 8 atoms, has ended with its GPU lost
    // since the split exists, for a cause that is not known, and members of that operator run as they did before.
    int kgrp = 1;
    if (extras && path == 3 && op.kind != OPEVO_CONV2D && ksteps % 2 == 0 && TM * TN <= 2 * 32 * 32 && ksteps * BK > 256) {
        const int64_t nw = WM * WN, stage = (BM + BN) * BK * 2, per = stage / (1024 * nw), wgs = n1 * m1 * b1;
        const bool pays = (nw == 1 && wgs <= 256 && ksteps >= 8) ||
                          (nw == 2 && wgs <= (stage <= 8192 ? 256 : 128) && stage <= 12288 && ksteps >= 16) ||
                          (nw == 4 && wgs <= 128 && stage <= 8192 && ksteps >= 32);
        // (the ring of both groups within the LDS, the sum of one of them within the ring, the loads in flight countable)
        for (int st = std::min(4, nstage_dlds); pays && st >= 2 && kgrp == 1; --st)
            if (2 * st * stage <= kMaxLds && nw * TM * TN * 4 <= 2 * st * stage && (2 * st - 2) * per <= 63 &&
                !(dlds_atom16 && BK % 64 != 0 && st % 2 != 0)) { kgrp = 2; nstage_dlds = 2 * st; out.extra_waves = true; }
    }
    // Grids of direct-to-LDS MatMul / BMM members that do not fit the chip at once, with eight waves or fewer on a compute unit: a ring of fewer stages leaves
    // room for more workgroups, which hide a slab's latency as well as the slabs ahead do.  The most stages with which the grid does fit: 88 drawn members 0.91 - 1.46x,
    // 1.12x in the geometric mean, 113 random ones 0.85 - 1.64x, 1.22x, three below 0.98 (1040 workgroups of two waves, 128 x 64, five slabs of 32: 11.7 -> 12.7 us).
    // With two waves or fewer on a compute unit, if it does not fit with any, the most stages that give it more: 20 drawn members 1.07 -
    // 1.40x, 1.22x (4544 x 3328 x 2112 in 64 x 128, two waves: 143 -> 104 us).  Three and more waves in grids that do
    // not fit in any case: 0.84 - 1.17x, 1.04x; those keep the ring.  So do members on 16x16x32 atoms: 30 drawn ones 0.59 - 1.76x, 1.14x, the slow ones (5120 x 1920 x 4096 in
    // 128 x 128, two waves, 115 -> 196 us; 5504 x 1536 x 1024 in 128 x 256, eight waves, 33 -> 40) with no line around them yet.
    if (path == 3 && kgrp == 1 && op.kind != OPEVO_CONV2D && !dlds_atom16) {
        const int64_t nw = WM * WN, stage = (BM + BN) * BK * 2, wgs = n1 * m1 * b1;
        auto resident = [&](int st) { return std::min<int64_t>(kMaxLds / (st * stage), 32 / nw); };
        const int64_t had = resident(nstage_dlds);
        if (wgs > 256 * had && had * nw <= 8) {
            int st = nstage_dlds;
            while (st > 2 && wgs > 256 * resident(st)) --st;
            if (wgs > 256 * resident(st) && had * nw <= 2)
                for (st = nstage_dlds; st > 2 && (resident(st) == had || resident(st) * nw < 4); --st) {}
            if (wgs <= 256 * resident(st) || (had * nw <= 2 && resident(st) > had)) nstage_dlds = st;
        }
    }
    // fp32 MatMul / BMM members with two stages, workgroup tiles of 32 or 64 rows and columns and long reductions: the template that takes values apart for the bf16
    // matrix pipes, its waves sharing the reduction, where the fp32 atoms are slower.  Up to 512 workgroups, which leave the fp32 atoms' members few waves a compute unit, from K = 320
    // on: 50 drawn operators 0.97 - 2.7x against the fastest of their fp32 members (slabs of 16, 32, 64, every division of the tile), 1.46x in the geometric mean.  On more workgroups the fp32
    // atoms' other workgroups hide what sharing the reduction does: K of 320 - 1024 0.81 - 1.1x (1792 x 2528 x 320 in 64 x 32 35.4 -> 43.3 us, 1344 x 2400 x 352 29.8 -> 36.2),
    // above 0.88 - 1.25x against the fastest and 0.89 - 1.54x, 1.2x in the mean, against 20 random ones: from 1056 on.  64 x 64 tiles, whose fp32 members read least: K of 448 - 864 0.86 - 1.0x
    // (512 x 192 x 544 11.8 -> 13.8), 896 - 1600 0.99 - 1.26x up to 512 workgroups; on more 704 0.98x, 768 - 1504 1.02 - 1.12x.  64 x 64
    // tiles with the first operand transposed need more registers than there are.  Batches on more than 400 workgroups, whose operands few tiles share, are bound by
    // bytes as much as by the pipes: 342 x (32 x 64 x 896), transposed, 23.9 -> 27.4, 250 x (128 x 64 x 704) 31.2 -> 34.4, 12 such members 0.87 - 1.17x, 0.99x; up to 400
    // 30 random ones in smaller tiles 1.06 - 2.9x, 15 of 64 x 64 0.98 - 1.64x.  69 further random members of what these lines leave, against the fp32 atoms 1.04 - 2.9x.
    // Eight waves instead of four where a compute unit has one workgroup at most and each wave still gets 88 steps: 44 drawn members 0.96 - 1.19x, 1.07x in the geometric
    // mean (416 x 320 x 704 in 32 x 64 10.8 -> 11.2 us, 64 x 64 x 1248 batches in 32 x 32 12.1 -> 10.2).
    int f32_kw = 0;
    const int64_t f32_wgs = n1 * m1 * b1, f32_least = BM * BN == 64 * 64 ? (f32_wgs <= 512 ? 896 : 768) : f32_wgs <= 512 ? 320 : 1056;
    if (extras && path == 4 && op.kind != OPEVO_CONV2D && flagv && ksteps > 1 && ksplit == 1 && subm * subn == 1 && WM * WN <= kMaxThreads / 64 &&
        (BM == 32 || BM == 64) && (BN == 32 || BN == 64) && !(op.trans_a && BM * BN == 64 * 64) && op.K % 32 == 0 && op.K >= f32_least &&
        (op.kind == OPEVO_MATMUL || f32_wgs <= 400) && op.M < (1 << 22) && op.N < (1 << 22) && op.K < (1 << 22) &&         // (a lane's byte offsets within 32 bits)
        valid_without_extras(op, variant, cfg)) {
        f32_kw = f32_wgs <= 256 && op.K >= 704 ? 8 : 4;
        out.extra_waves = true;
        WM = 1; WN = f32_kw; TM = BM; TN = BN; TMacc = TM; TNacc = TN; FM = std::gcd(FM, TM); FN = std::gcd(FN, TN);
    }
    const bool b_kmajor = path == 3 && (b_packed || op.kind == OPEVO_CONV2D);
    const bool nhwc = nhwc_ok && (path == 1 || path == 2 || path == 3);
    // a transposed first operand is staged by the MFMA templates like B (rows of 8 along M), so it
    // needs M % 8 == 0 and LDS staging; other members run on the scalar template
    if (op.trans_a && (path == 1 || path == 2) && (op.M % 8 != 0 || !stage_lds)) path = 0;

    int64_t NT, nwr = WM * WN * patch_kw;   // nwr: waves the workgroup really runs
    if (four_level) {
        if (path == 0) nwr = std::min<int64_t>(nwr, kMaxThreads / 64);   // the scalar template deals outputs round-robin to any number of threads
        else while (path != 5 && path != 6 && path != 7 && nwr > kMaxThreads / 64) {      // largest divisor of WM * WN that fits
            int64_t best = 1;
            for (int64_t dv = kMaxThreads / 64; dv >= 1; --dv) if ((WM * WN) % dv == 0) { best = dv; break; }
            nwr = best;
        }
        NT = 64 * nwr;
    }
    else {
        NT = ((BM * BN + 63) / 64) * 64;
        if (NT > 256) NT = 256;
    }
    int64_t acc = (path == 0) ? (BM * BN + NT - 1) / NT : (TMacc * TNacc) / 64 * (f32_kw ? 2 : 1);
    const int nstage = path == 7 ? 1 : path == 6 ? rg.stages : path == 5 ? patch_stages : path == 3 ? nstage_dlds : (path != 0 && flagv && ksteps > 1) ? 2 : 1;
    int64_t lds = 0;
    if (path == 0) lds = (BM * BK + BK * BN) * 4;
    else if (path == 4 && op.kind == OPEVO_CONV2D) {
        const int64_t a_rows = (WM - 1) * TM + TMacc, b_cols = ((WN - 1) * TN + TNacc + 3) / 4 * 4;   // with the overhang
        lds = nstage * (a_rows * (BKP + 4) + BKP * (b_cols + 4)) * 4;
    }
    else if (path == 4 && f32_kw) lds = f32_kw * BM * std::max<int64_t>(op.trans_a ? 0 : 64, BN) * 4;
    else if (path == 4) lds = nstage * ((op.trans_a ? BK * (BM + 4) : BM * (BK + 4)) + BK * (BN + 4)) * 4;
    else if (path == 3) lds = nstage * (anr + (b_kmajor ? bnr : BN)) * BK * 2;
    else if (path == 5 && strip.rows) lds = strip.lds;
    else if (path == 5)   // the stages, or (more than one wave per tile) one atom of every wave if that is more
        lds = std::max<int64_t>(nstage * (nb2 * patch_image * (patch_cs + 8) + op.hk * op.wk * BM * patch_cs + 64) * 2,
                                patch_kw > 1 ? nwr * (patch_atom == 32 ? 4 : 1) * 1024 : 0);
    else if (path == 6) lds = rg.lds;
    else if (path == 7) lds = rows.lds;
    else if (stage_lds) lds = nstage * (BM + BN) * (BKP + kPad) * 2 + (ragged ? 16 * (BKP + kPad) * 2 : 0);   // overhang rows stay inside the allocation

    p.path = path;
    const int64_t n_blocks = n1 * m1 * b1;
    if (linear) { p.grid[0] = int32_t(n_blocks > INT32_MAX ? INT32_MAX : n_blocks); p.grid[1] = 1; p.grid[2] = 1; }
    else { p.grid[0] = int32_t(n1); p.grid[1] = int32_t(m1); p.grid[2] = int32_t(b1); }
    if (rows.persist > 0) p.grid[0] = rows.persist;   // workgroups that take several boxes each
    p.block = int32_t(NT > INT32_MAX ? INT32_MAX : NT * kgrp);
    p.lds_bytes = int32_t(lds > INT32_MAX ? INT32_MAX : lds);
    out.static_lds = path == 3 ? p.lds_bytes : int32_t(rows.beside);
    p.acc_per_lane = int32_t(acc > INT32_MAX ? INT32_MAX : acc);
    p.tile[0] = int32_t(BM); p.tile[1] = int32_t(BN); p.tile[2] = int32_t(BK);
    p.wave_tile[0] = int32_t(four_level ? TM : BM); p.wave_tile[1] = int32_t(four_level ? TN : BN);
    p.sub_tiles[0] = int32_t(subm); p.sub_tiles[1] = int32_t(subn);
    p.wave_passes = int32_t(four_level && nwr > 0 && path != 5 && path != 6 && path != 7 ? (WM * WN) / nwr : 1);

    // ---- black-box constraints made explicit: such members get fitness 0 (Sec. 4.2)
    if (NT > kMaxThreads) invalid(p, "%ld threads per workgroup > %ld", long(NT), long(kMaxThreads));
    else if (acc > kMaxAcc) invalid(p, "%ld accumulators per lane > %ld", long(acc), long(kMaxAcc));
    else if (lds + ((path == 0 || subm * subn * ((WM * WN) / std::max<int64_t>(nwr, 1)) > 1) ? 16 : 0) > kMaxLds)   // the deadline flag word of the scalar template and of folded members
        invalid(p, "%ld bytes of LDS > %ld", long(lds), long(kMaxLds));
    else if (!linear && (m1 > 65535 || b1 > 65535)) invalid(p, "grid y/z %ld x %ld > 65535", long(m1), long(b1));
    else if (linear && n_blocks > INT32_MAX) invalid(p, "%ld workgroups in a one-dimensional grid", long(n_blocks));
    else if (path == 4 && !f32_kw) {
        const int64_t chunks = op.kind == OPEVO_CONV2D ? (BM * (BKP / 4) + NT - 1) / NT + (BKP * ((BN + 3) / 4) + NT - 1) / NT
                                                       : (BM * (BK / 4) + NT - 1) / NT + (BK * (BN / 4) + NT - 1) / NT;
        if (chunks * 4 > 256) invalid(p, "%ld staging registers per lane > 256", long(chunks * 4));
    }
    else if (path != 0 && path != 3 && path != 4 && path != 5 && path != 6 && path != 7 && stage_lds) {
        // register budget of the slab in flight: 16-byte pieces per thread
        const int64_t a_chunks = op.trans_a ? 8 * (((BK / 8) * (BM / 8) + NT - 1) / NT) : (BM * (BKP / 8) + NT - 1) / NT;
        const int64_t b_chunks = (op.kind == OPEVO_CONV2D) ? (BN * (BKP / 8) + NT - 1) / NT
                                                           : 8 * (((BK / 8) * (BN / 8) + NT - 1) / NT);
        if ((a_chunks + b_chunks) * 4 > 256)
            invalid(p, "%ld staging registers per lane > 256", long((a_chunks + b_chunks) * 4));
    }

    out.tmpl = path == 0 ? "gemm_scalar" : path == 3 ? "gemm_mfma_dlds" : path == 4 ? (f32_kw ? "gemm_f32_split" : "gemm_mfma_f32") : path == 5 ? (strip.rows ? "conv_strip" : "conv_patch") : path == 6 ? "gemm_ragged" : path == 7 ? "conv_rows" : "gemm_mfma";
    // One symbol per configuration, so profiles list each instantiated kernel on its own line.  Templates that take the workgroup tile alone and divide it by
    // themselves make one program of all configurations with that tile (box): they are named by it, and given no constant that they do not read, so
    // that the program is compiled once.
    const bool whole = f32_kw || rg_kw;             // every wave has the whole tile
    {
        std::ostringstream nm;
        nm << "opevo_" << (op.kind == OPEVO_MATMUL ? "mm" : op.kind == OPEVO_BMM ? (op.trans_a ? "bmmt" : "bmm") : "conv");
        if (whole) {
            nm << (f32_kw ? "_split_" : "_shared_") << BM << "_" << BN << "_" << (f32_kw ? f32_kw : rg_kw) << "_" << binner;
            if (linear) nm << "_" << order[0] << order[1] << order[2] << "_" << group;
        } else if (strip.rows) {
            nm << "_strip_" << BM << "_" << nb2 << "_" << BH << "_" << BW << "_" << strip.cs << "_" << strip.wm << "_" << strip.rows << "_" << strip.kw;
            flagv = 0; FM = FN = 1;
        } else nm
           << (variant == OPEVO_TILE4P ? "p" : variant == OPEVO_TILE4K ? "k" : variant == OPEVO_TILE4C ? "c" : variant == OPEVO_TILE4T ? "t" : variant == OPEVO_TILE4A ? "a" : variant == OPEVO_TILE4L ? "l" : four_level ? "4" : "2");
        int width = 0;
        for (const auto &d : descs) width += d.type == OPEVO_FACTOR ? d.nu : d.type == OPEVO_PERMUTATION ? d.n_values : 1;
        for (int i = 0; i < width && !whole && !strip.rows; ++i) nm << "_" << cfg[i];
        out.kernel_name = nm.str();
    }
    D << "-DKERNEL_NAME=" << out.kernel_name << " ";
    D << "-DOP=" << op.kind << " -DIN_DTYPE=" << op.dtype << " -DM=" << op.M << " -DN=" << op.N
      << " -DK=" << op.K << " -DBM=" << BM << " -DBN=" << BN << " -DNT=" << NT << " -DBATCH_INNER=" << binner << " -DA_TRANS=" << (op.trans_a ? 1 : 0);
    if (!whole) D << " -DBK=" << BK << " -DKSTEPS=" << ksteps << " -DFLAG=" << flagv;
    if (path != 0 && !whole) {
        D << " -DATOM=" << (path == 7 ? rows.atom : path == 5 ? patch_atom : (path == 2 || path == 6 || dlds_atom16) ? 16 : 32) << " -DWM=" << WM << " -DWN=" << WN << " -DTM=" << TM
          << " -DTN=" << TN << " -DFM=" << FM << " -DFN=" << FN << " -DPAD=" << kPad
          << " -DNSTAGE=" << nstage << " -DNSTG=" << nstage << " -DSTAGE_LDS=" << (stage_lds ? 1 : 0);
        if (nwr != WM * WN && path != 5) D << " -DNWR=" << nwr;
    }
    if (path == 7) D << " -DWKP=" << rows.wkp << " -DMI=" << rows.mi << " -DNI=" << rows.ni << " -DLDS_BYTES=" << lds << " -DPERSIST=" << rows.persist << " -DNBOX=" << n1 << " -DBESIDE=" << rows.beside;
    if (rg_kw) D << " -DKWAVES=" << rg_kw << " -DLDS_BYTES=" << lds << " -DMINW=" << rg.min_waves;
    else if (path == 6) D << " -DKS=" << rg.ks << " -DNSL=" << rg.slabs << " -DMI=" << rg.mi << " -DNI=" << rg.ni << " -DLDS_BYTES=" << lds << " -DDEPTH=" << rg.depth << " -DMINW=" << rg.min_waves;
    if (subm * subn > 1) {
        D << " -DSUBM=" << subm << " -DSUBN=" << subn;
    }
    if (op.kind == OPEVO_CONV2D) {
        D << " -DCIN=" << op.cin << " -DHIN=" << op.hin << " -DWIN=" << op.win << " -DHK=" << op.hk
          << " -DWK=" << op.wk << " -DSTRIDE=" << op.stride << " -DPAD_CONV=" << op.pad
          << " -DHOUT=" << op.hout << " -DWOUT=" << op.wout << " -DNB2=" << nb2 << " -DBH=" << BH
          << " -DBW=" << BW << " -DH1=" << h1 << " -DW1=" << w1 << " -DBKP=" << BKP;
        // the MFMA template gathers the image through a compile-time table of tap offsets where its
        // fields are wide enough (byte offsets into the image tensor in 32 bits, padded image
        // coordinates in 15) and the table stays small (8 bytes per position of the reduction walk)
        const bool table = path != 0 && op.b_elems() < (int64_t(1) << 31) && op.hin + 2 * op.pad < 32768 &&
                           op.win + 2 * op.pad < 32768 && op.hk < 32768 && op.wk < 32768 && ksplit * ksteps * BKP <= 8192 && !nhwc && path != 7;
        if (path != 0) D << " -DCONV_TABLE=" << (table ? 1 : 0);
        if (nhwc) D << " -DCONV_NHWC=1";
    }
    if (tap_box)
        D << " -DTAP_BOX=1 -DCI_O=" << box[0] << " -DCI_I=" << box[1] << " -DHK_O=" << box[2] << " -DHK_I=" << box[3]
          << " -DWK_O=" << box[4] << " -DWK_I=" << box[5];
    if (path == 5 && strip.rows)
        D << " -DCS=" << strip.cs << " -DPWP=" << strip.pitch << " -DKW=" << strip.kw << " -DMI=" << strip.mi << " -DR=" << strip.rows << " -DMINW=" << strip.min_waves
          << " -DLDS_BYTES=" << lds;
    else if (path == 5) D << " -DCS=" << patch_cs << " -DPWP=" << patch_row << " -DIPIX=" << patch_image << " -DKW=" << patch_kw << " -DLDS_BYTES=" << lds;
    if (b_kmajor) D << " -DB_KMAJOR=1 -DBNR=" << bnr;
    if (path == 3 && anr != BM) D << " -DANR=" << anr;
    // ragged: the places of pieces kept where they fit, or may fit; else worked out where they are needed, for every slab anew if the kernel spills
    // otherwise (one in 100 members; transposed first operands on eight waves of 3 x 7 to 3 x 9 atoms always do)
    if (path == 6 && !rg_kw) {
        const bool spills = op.trans_a && rg.keep != 1 && rg.wm * rg.wn >= 8 && rg.mi >= 3 && rg.mi * rg.ni >= 20;
        out.tries.clear();
        if (rg.keep == 1 || (rg.keep == 2 && !spills)) out.tries.push_back(" -DKEEP=1");
        if (rg.keep != 1 && !spills) out.tries.push_back(" -DKEEP=0");
        out.tries.push_back(" -DKEEP=0 -DFRESH=1");
    }
    // The kernel tensor's rows through the LDS, and straight from memory if the kernel spills so (one of 695 drawn members: 33 x 3 x 224 x 224 * 128 x 3 x 11 x 11, stride 4, on the
    // register-staged template instead 295 us, 67 so).  What it would have beside the patch is counted all the same.
    if (path == 7) {
        out.tries.clear();
        if (rows.stage) out.tries.push_back(rows.stage == 1 ? " -DSTAGE_A=1" : " -DSTAGE_A=2");
        out.tries.push_back(" -DSTAGE_A=0");
    }
    // A patch: two slabs of global loads in flight instead of one where a slab's MFMAs are too few to cover its loads: kernel tensors of
    // one tap, and up to nine taps on waves that share their tiles' steps in grids of one workgroup per compute unit, in slabs of up to 32 channels.  One tap: 163 random
    // members 0.89 - 1.58x, 1.05x in the geometric mean (88 x 256 x 27 x 27 * 128 x 256 33.6 -> 30.4 us, 6 x 256 x 27 x 27 * 192 x 256 8.2 -> 6.5); shared tiles 126
    // members 0.94 - 1.16x, 1.05x (40 x 256 x 7 x 7 * 96 x 256 x 3 x 3 12.2 -> 10.7).  Slabs of 64 channels have MFMAs enough, and their second set of registers costs resident
    // workgroups: 25 members 0.75 - 1.07x, 0.95x (5 x 256 x 56 x 56 * 192 x 256 on 1680 workgroups of one wave, 232 -> 422 registers, 18.9 -> 25.4).  25 taps 0.93 - 1.13x, five larger grids 0.77 - 1.06x,
    // 22 members that share nothing 0.85 - 1.03x, 0.94x.
    if (path == 5 && !strip.rows && nstage == 2 && ksteps >= 3 && patch_cs <= 32 && (op.hk * op.wk == 1 || (patch_kw > 1 && op.hk * op.wk <= 9 && n_blocks <= 256)))
        out.tries = {" -DSLABS_AHEAD=2", ""};
    // fp32, two stages: the pipelined slab loop, but for short reductions on a full chip, where the other workgroups cover a
    // slab's latency and the registers are better spent on them (a batch of 960 of 128 x 64 x 128 with the first operand transposed:
    // 960 x 4 waves, 4 slabs, 27.0 us without and 29.9 with; 132 x 64 x 224 x 128, 924 x 2 waves, 2 slabs, 16.2 and 13.9).  Against the
    // plain loop 13 MatMul / BMM members on slabs of 8 are 1.00 - 1.46 times as fast, 70 members on longer slabs 0.97 - 1.56 and one (4 slabs of
    // 24, 42 x 2 waves) 0.94.
    // Slabs of a single group of 8 have nothing to read ahead.  Convolutions on them, which gather value by value, and short
    // reductions on a full chip have the plain loop with the second operand read step by step (8 x 64 x 28 x 28 * 64 x 64 x 3 x 3 as 112 x 1 waves 77.5 us so and
    // 82.0 pipelined, as 112 x 7 waves 54.8 and 61.1, on slabs of 2 as 32 x 1 waves 1020 and 1139; 2048 x 2048 x 128, 1024 x 2 waves, 15.7 and 17.5; four other
    // convolutions between 0.7 % slower and 2 % faster).
    if (path == 4 && nstage == 2 && !f32_kw) {
        const bool full_chip = n_blocks * nwr >= 2048;
        if (BKP == 8 && (op.kind == OPEVO_CONV2D || (full_chip && ksteps * BKP <= 128))) out.tries = {" -DSTEP_READS=1", " -DPIPELINED=1", ""};
        else if (!(full_chip && ksteps < 8)) out.tries = {" -DPIPELINED=1", ""};
    }
    // fp32, short reductions: outputs that the eight L2s (32 MiB) would hold and write back when the kernel ends are stored past them.  44 further
    // MatMul / BMM members of K <= 224 with outputs of 2 - 32 MiB, drawn after the rule was made, 1.00 - 1.28x, 1.04x in the geometric mean (727 x (128 x 64 x 64)
    // 16.1 -> 13.1 us, 448 x 2112 x 192 6.87 -> 6.64); smaller outputs 0.96 - 1.06x, larger ones 0.95 - 1.07x; 42 further ones with an elementwise pass over the
    // output after them 1.01x for the two together (0.94 - 1.13), 1.03x alone; K of 256 to 6208 0.91 - 1.02x (mostly 1.00).  Rows of 64 or of any number of bytes (16-bit
    // inputs on 16 x 16 atoms, ragged tiles) 0.59 - 1.20x without a line between them: those stay with ordinary stores.
    const int64_t out_bytes = op.c_elems() * 4;
    if (path == 4 && !f32_kw && op.kind != OPEVO_CONV2D && ksplit == 1 && op.K <= 224 && out_bytes >= (int64_t(2) << 20) && out_bytes <= (int64_t(32) << 20)) D << " -DNT_OUT=1";
    if (f32_kw) D << " -DKW=" << f32_kw << " -DLDS_BYTES=" << lds << " -DMINW=2";
    if (kgrp > 1) D << " -DKGRP=" << kgrp;
    if (kunroll) D << " -DKUNROLL=" << kunroll;
    if (ksplit > 1) D << " -DKSPLIT=" << ksplit;
    out.zero_bytes = ksplit > 1 ? op.c_elems() * 4 : 0;
    out.prepass = nhwc ? 1 : (b_kmajor && op.kind == OPEVO_MATMUL) ? 2 : 0;
    std::string walked;
    if (!linear && four_level && op.kind != OPEVO_CONV2D && ksplit == 1 && n_blocks < (int64_t(1) << 30))
        if (const int walk = xcd_walk(op, n1, m1, b1, BM * subm, BN * subn, binner, lds > 0 ? kMaxLds / lds : 8, path != 0)) {
            std::ostringstream W;
            W << " -DXCD_WALK=" << walk << " -DGRID_N1=" << n1 << " -DGRID_M1=" << m1 << " -DGRID_B1=" << b1;
            // A single row of tiles is number 0, which the natural order's code does not know.  Members that read their fragments straight from global memory,
            // several batches a workgroup, in 9 to 15 steps stand where it decides whether the compiler unrolls all steps; unrolled over two batches every
            // load was waited for by itself (64, 100, 190, 512 x (128 x 128 x 192) in 128 x 32 8.3, 12.2, 17.4, 31.7 us in the natural order, 14.0, 14.5,
            // 18.1, 36.3 walked, 8.5, 8.8, 12.3, 23.2 walked without that knowledge; with one batch a workgroup, or on 16-row atoms, it is a gain).
            if (path == 1 && !stage_lds && binner > 1 && m1 == 1 && op.K / 16 > 8 && op.K / 16 < 16) W << " -DROW_UNKNOWN=1";
            walked = W.str();
        }
    if (!walked.empty()) {   // a member that spills with the walk, whatever else is tried, is built in the natural order
        const std::vector<std::string> natural = out.tries;
        for (std::string &t : out.tries) t += walked;
        out.tries.insert(out.tries.end(), natural.begin(), natural.end());
    }
    if (linear)
        D << " -DGRID_LINEAR=1 -DGRID_N1=" << n1 << " -DGRID_M1=" << m1 << " -DGRID_B1=" << b1 << " -DORDER0=" << order[0]
          << " -DORDER1=" << order[1] << " -DORDER2=" << order[2] << " -DGROUP=" << group;
    out.defines = D.str();
    return OPEVO_OK;
}

}  // namespace opevo

extern "C" {

int opevo_op_create(int kind, const int64_t *dims, int n_dims, int in_dtype, opevo_op **out)
{
    if (!dims || !out) return fail(OPEVO_E_ARG, "op_create: NULL argument");
    if (in_dtype < OPEVO_F32 || in_dtype > OPEVO_F16) return fail(OPEVO_E_ARG, "op_create: unknown dtype %d", in_dtype);
    opevo_op op;
    if (kind == OPEVO_BMM_TA) { kind = OPEVO_BMM; op.trans_a = true; }
    op.kind = kind; op.dtype = in_dtype;
    const int need = kind == OPEVO_MATMUL ? 3 : kind == OPEVO_BMM ? 4 : kind == OPEVO_CONV2D ? 9 : -1;
    if (need < 0) return fail(OPEVO_E_ARG, "op_create: unknown operator kind %d", kind);
    if (n_dims != need) return fail(OPEVO_E_ARG, "op_create: operator needs %d dims, got %d", need, n_dims);
    for (int i = 0; i < n_dims; ++i) {
        const bool may_be_zero = (kind == OPEVO_CONV2D && i == 8);   // padding
        if (dims[i] < (may_be_zero ? 0 : 1) || dims[i] > (int64_t(1) << 30))
            return fail(OPEVO_E_ARG, "op_create: dims[%d] = %lld out of range", i, (long long)dims[i]);
    }
    if (kind == OPEVO_MATMUL) { op.M = dims[0]; op.N = dims[1]; op.K = dims[2]; }
    else if (kind == OPEVO_BMM) { op.batch = dims[0]; op.M = dims[1]; op.N = dims[2]; op.K = dims[3]; }
    else {
        op.nimg = dims[0]; op.cin = dims[1]; op.hin = dims[2]; op.win = dims[3];
        op.M = dims[4]; op.hk = dims[5]; op.wk = dims[6]; op.stride = dims[7]; op.pad = dims[8];
        const int64_t sh = op.hin + 2 * op.pad - op.hk, sw = op.win + 2 * op.pad - op.wk;
        if (sh < 0 || sw < 0) return fail(OPEVO_E_ARG, "op_create: kernel larger than the padded image");
        op.hout = sh / op.stride + 1;    // App. B.3
        op.wout = sw / op.stride + 1;
        op.K = op.cin * op.hk * op.wk;
        op.N = op.nimg * op.hout * op.wout;
    }
    if (double(op.batch) * double(op.M) * double(op.N) > 4.0e18 || op.a_elems() < 0 || op.b_elems() < 0)
        return fail(OPEVO_E_ARG, "op_create: tensor too large");
    *out = new (std::nothrow) opevo_op(op);
    return *out ? OPEVO_OK : fail(OPEVO_E_ARG, "out of memory");
}

int opevo_op_destroy(opevo_op *op) { delete op; return OPEVO_OK; }

int opevo_op_flops(const opevo_op *op, double *flops)
{
    if (!op || !flops) return fail(OPEVO_E_ARG, "op_flops: NULL argument");
    *flops = op->flops();
    return OPEVO_OK;
}

int opevo_op_bytes(const opevo_op *op, double *bytes)
{
    if (!op || !bytes) return fail(OPEVO_E_ARG, "op_bytes: NULL argument");
    *bytes = double(op->a_elems() + op->b_elems()) * op->elem_size() + double(op->c_elems()) * 4.0;
    return OPEVO_OK;
}

int opevo_op_sizes(const opevo_op *op, int64_t *a_elems, int64_t *b_elems, int64_t *c_elems)
{
    if (!op) return fail(OPEVO_E_ARG, "op_sizes: NULL argument");
    if (a_elems) *a_elems = op->a_elems();
    if (b_elems) *b_elems = op->b_elems();
    if (c_elems) *c_elems = op->c_elems();
    return OPEVO_OK;
}

int opevo_op_space(const opevo_op *op, int variant, opevo_space **out)
{
    if (!op || !out) return fail(OPEVO_E_ARG, "op_space: NULL argument");
    std::vector<opevo_param_desc> descs;
    if (int rc = op_param_descs(*op, variant, descs)) return rc;
    return opevo_space_create(descs.data(), int(descs.size()), out);
}

int opevo_kernel_plan(const opevo_op *op, int variant, const int32_t *cfg, opevo_plan *plan)
{
    if (!op || !cfg || !plan) return fail(OPEVO_E_ARG, "kernel_plan: NULL argument");
    Decoded d;
    if (int rc = decode(*op, variant, cfg, d)) return rc;
    *plan = d.plan;
    return OPEVO_OK;
}

int opevo_kernel_defines(const opevo_op *op, int variant, const int32_t *cfg, char *buf, size_t cap)
{
    if (!op || !cfg || !buf) return fail(OPEVO_E_ARG, "kernel_defines: NULL argument");
    Decoded d;
    if (int rc = decode(*op, variant, cfg, d)) return rc;
    const std::string s = d.tmpl + ": " + d.defines + d.tries.front();
    if (s.size() + 1 > cap) return fail(OPEVO_E_ARG, "kernel_defines: buffer too small (%zu needed)", s.size() + 1);
    std::memcpy(buf, s.c_str(), s.size() + 1);
    return OPEVO_OK;
}

}  // extern "C"
