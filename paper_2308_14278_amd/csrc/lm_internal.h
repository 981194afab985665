// lm_internal.h -- layouts shared by the host code and the gfx950 kernels of
// liblensmap (not part of the public ABI).
#pragma once
#include <stdint.h>

#define LM_WG 256          // threads per workgroup: 4 waves of 64
#define LM_WAVES 4
#define LM_LENS_CAP 256    // direct sum: lenses staged per wave per block (the summation block)
// Kernel value of LM_PREC_MIXED_CENTRED: FP32 near sums of each near lens's
// deflection change from the level-2 cell centre, whose near-lens deflection
// is taken in FP64 (n0 below).
constexpr int kPrecCentred = 4;
// The `terms` the direct scheme's shooting kernels are asked for with: 1, or for lists
// of more than one block of lenses this.
constexpr int kLongList = 2;
constexpr int lm_direct_terms(int64_t nlens) { return nlens > LM_LENS_CAP ? kLongList : 1; }

// LDS layouts of the interpolated-scheme shooting kernels, the tuner's third
// axis besides rays per lane and tile size: lenses per LDS table block (the
// wave-shared dx^2, m dx table), uint32 bins of the workgroup's LDS window
// (the histogram tile), near lenses staged per wave per block.  With 16 rays
// per lane and FP32 sums each fits 40 KiB per workgroup (four per CU).  Layout
// 0 serves every kernel; the others are built for the FP32 rebased path with
// P = 4 and 8 or 16 rays per lane.  Results never depend on the layout.
#define LM_LAYOUTS 4
static constexpr int kLayTab[LM_LAYOUTS] = {16, 8, 32, 16};
static constexpr int kLayWin[LM_LAYOUTS] = {7040, 8064, 5000, 7552};
static constexpr int kLayNear[LM_LAYOUTS] = {64, 64, 64, 32};

// Table entries per (column, lens) of a precision's wave-shared LDS table: dx^2
// and m dx, or for the centred sums dx^2, c_r dx and c_i dx.
constexpr int tab_width(int prec) { return prec == kPrecCentred ? 3 : 2; }

// Window bins of a shooting kernel: the layout's, less what the wider table of
// the centred sums takes (rays_per_lane columns per lens and wave); or what the
// direct scheme's lens blocks leave of 40 KiB.  Either way the workgroup keeps to
// the layout's LDS budget, four to a CU (the direct scheme on layout 0's window
// took 43.5 KiB: three).
constexpr int window_bins(int scheme, int prec, int layout, int rays_per_lane)
{
    return scheme == 0 ? 6080
                       : kLayWin[layout] - (prec == kPrecCentred
                                                ? LM_WAVES * kLayTab[layout] * rays_per_lane
                                                : 0);
}

// Allocation-free peak statistics: limits and layout of the per-device scratch
// array (tracks, first columns of the bins, two histograms, the count of finished
// workgroups, the bins' results; each part 256-byte aligned).  LM_SCRATCH_COLS
// is the entry point's limit on map columns; nothing of the array is per column.
#define LM_SCRATCH_TRACKS 8192
#define LM_SCRATCH_COLS (1 << 20)
#define LM_SCRATCH_BINS 4096
#define LM_SCRATCH_OFF_BINS (4 * LM_SCRATCH_TRACKS)
#define LM_SCRATCH_OFF_HIST (LM_SCRATCH_OFF_BINS + (4 * (LM_SCRATCH_BINS + 1) + 255) / 256 * 256)
#define LM_SCRATCH_OFF_DONE (LM_SCRATCH_OFF_HIST + 16 * LM_SCRATCH_BINS)
#define LM_SCRATCH_OFF_OUT (LM_SCRATCH_OFF_DONE + 256)
#define LM_SCRATCH_BYTES (LM_SCRATCH_OFF_OUT + 16 * LM_SCRATCH_BINS)
#define LM_MAX_DEVICES 64

// Taylor coefficients of one level-2 cell: a_0 in FP64 (it carries the large
// far-field deflection of the cell centre), a_1..a_6 in FP32 (they multiply
// offsets of at most half a cell); and for the centred near sums the
// deflection of the cell centre by its near lenses, FP64, NaN when a near lens
// lies within twice the cell's half-diagonal of the centre.  80 bytes per cell.
struct LmCoef {
    double a0r, a0i;
    double n0x, n0y;
    float a[12];  // (re, im) of a_1 .. a_6
};

// Everything a kernel needs about one map and one shot rectangle.
struct LmDesc {
    // ray lattice and macro mapping (FP64)
    double x0, y0, dx, dy;
    double mx, my;                 // linear: 1-kappa-gamma+kappa_star, 1-kappa+gamma+kappa_star;
                                   // fold: kappa_star, 2(1-kappa0)+kappa_star
    double qx, qy;                 // fold: d_x/2, d_y (beta_x gains (qx theta_x + qy theta_y) theta_x)
    double bx0, by0, inv_sdx, inv_sdy;
    double sx0, sx1, sy0, sy1;     // rectangle of the -kappa_star sheet (sheet = 1)
    double kappa_star;
    // FP32 copies: half ray spacing as float-float (rebased arithmetic) and
    // plain values (the global-FP32 comparison path)
    float hxh, hxl, hyh, hyl;
    float x0f, y0f, dxf, dyf;
    float mxf, myf, bx0f, by0f;
    float inv_sdxf, inv_sdyf;
    int32_t snx, sny;
    int32_t fold;                  // 1: fold macro model
    int32_t sheet;                 // 1: the sheet covers [sx0, sx1] x [sy0, sy1]
    int32_t Q;                     // terms of the level-1 series (0: direct coefficients)
    int32_t nbx, nby;              // boxes of the level-1 series per level-1 cell side
    int32_t bx, by;                // level-2 cells per box side (the last box may be narrower)
    // scheme and work decomposition
    int32_t R, Kx, Ky, H;
    int32_t G;                     // level-2 cells per workgroup-tile side
    int32_t ncc;                   // column chunks per level-2 cell and workgroup
    int32_t cw;                    // columns per chunk
    int32_t nrb;                   // 64-row blocks per level-2 cell (R / 64)
    int32_t wx, wy;                // LDS window (pixels)
    int32_t nl1x, nl1y;            // padded level-1 grid (N1 + 2H per side)
    int64_t n1x, n1y;              // level-1 cells holding level-2 cells of the lattice
    int64_t nx, ny;                // lattice
    int64_t i0, j0, i1, j1;        // shot rectangle [i0,i1) x [j0,j1)
    int64_t ncx, ncy;              // level-2 cells of the lattice
    int64_t tcx0, tcy0, ntx, nty;  // workgroup tiles covering the rectangle
    int64_t ntiles;
    int64_t tile0;                 // first tile of a k_shoot_map launch
    int64_t nlens;
    // lenses: sorted by level-1 cell for the interpolated scheme
    const double* lx;
    const double* ly;
    const double* lmd;
    const float* lxf;
    const float* lyf;
    const float* lmf;
    const int32_t* lI;             // level-1 cell of each lens (clamped)
    const int32_t* lJ;
    const int32_t* cell_start;     // CSR over the padded level-1 grid
    const LmCoef* coef;            // [ncy][ncx]
    double* l1exp;                 // [n1y nby][n1x nbx][Q] level-1 series per box, complex
    unsigned long long* counts;    // [sny][snx]
    unsigned long long* n_out;
    // workgroups that share a tile in a k_shoot_map launch (its grid's y size), each
    // with ncc column chunks of every cell
    int32_t split;
};

// How a launch for one map shares its tiles out: workgroups to a tile, columns per
// chunk of a cell, rays per lane.
struct LmSplit {
    int split, cw, nr;
};

// Tiles of a small rectangle are shared by several workgroups, each with shorter
// column chunks and, below 16 columns, fewer rays per lane: with one or two waves
// per SIMD a launch lasts as long as one wave's chain over its columns and lenses,
// which a split shortens.  A ray's sums do not depend on the split: the counts are
// the same.
//
// form: 0 direct, 1 FP32 near sums, 2 FP64; R, ncc, cw: rays a side, column chunks and
// columns per chunk of a cell; tiles of G x G cells (more than one: not split); ni x nj
// rays; list, longest: mean and longest list of lenses; cus: CUs.
//
// The split and the rays per lane are those of the least time in a model of the
// launch: a wave's steps of nr columns, each lens of the longest list taking `lat` ns
// alone or, with k waves on its SIMD, each of a mean list k times `issue` (lists
// counted `col` lenses longer, for starting and counting the columns), and 25 ns for
// each workgroup, whose window is cleared and flushed.  The figures are fits to
// launches of 4 to 2048 workgroups, among them (us, 1, 2 and 4 workgroups to a tile
// of 64 x 64 rays):
//   direct  250 x 190 rays,    30 lenses  20.1  14.9  12.3      300  87.0 55.0 38.1
//           1000 x 1000,       10         19.8  21.8  30.6      300  91.4 72.8 69.9
//           1400 x 1400,       10         26.0  30.6  49.8      300  122  115  125
//   FP32    1000 x 1000,       10 near    17.0  21.4  32.9      300  90.4 70.2 70.4
//           1400 x 1400,       10         21.6  29.9  51.7      300  101  103  126
//   FP64    1000 x 1000,       10         18.7  21.7  36.2      300  120  101  115
// and of 128 x 128 rays, 1, 2, 4 and 8 (FP32):
//           1000 x 1000,       10 near    29.6  20.0  16.9 21.1 300  323  168  91.7 70.8
//           2000 x 2000,       10         29.2  25.9  33.5 58.3 300  325  191  166  183
inline LmSplit lm_split(int form, int R, int ncc, int cw, int G, int64_t tiles, int64_t ni,
                        int64_t nj, double list, double longest, int cus)
{
    constexpr double lat[3][3] = {{254, 151, 98}, {255, 160, 115}, {360, 204, 139}};
    constexpr double issue[3][3] = {{125, 72, 40}, {114, 62, 33}, {237, 122, 71}};
    constexpr double col = 6.0;
    const auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const int64_t rows = up(nj < R ? nj : R, 64);  // row blocks in use
    LmSplit best{1, cw, 16};
    double least = 0.0;
    for (int s = 1; s == 1 || (G == 1 && cw % (4 * s) == 0 && s * tiles <= 8 * cus); s *= 2) {
        const int c = cw / s;
        const int64_t ncol = ni + 1 < c ? ni + 1 : c;  // (one more may make the first even)
        const int64_t chunks = up(ni < R ? ni : R, c);  // in use
        const int64_t units = rows * (chunks < ncc ? chunks : ncc);  // of a workgroup
        // waves per SIMD
        const double k = G > 1 ? 4.0
                               : (double)up(tiles * up(chunks, ncc), cus) *
                                     (double)(units < LM_WAVES ? units : LM_WAVES) / LM_WAVES;
        for (int q = 0; q < 3; ++q) {
            const int nr = 16 >> q;
            const double alone = lat[form][q] * (longest + col);
            // (long direct lists run two waves per SIMD at 16 rays per lane)
            const double each =
                q == 0 && form == 0 && longest > LM_LENS_CAP ? 165.0 : issue[form][q];
            const double shared = k * each * (list + col);
            const double t =
                (double)(up(units, LM_WAVES) * up(ncol, nr)) * (alone > shared ? alone : shared) +
                25.0 * (double)(s * tiles);
            // (a per cent of a model is worth no more workgroups or steps)
            if (least == 0.0 || t < 0.985 * least) {
                least = t;
                best = LmSplit{s, c, nr};
            }
        }
    }
    return best;
}

// Device lens arrays of a map (LmDesc's, writable).
struct LmLensArrays {
    double *lx, *ly, *lmd;
    float *lxf, *lyf, *lmf;
    int32_t *lI, *lJ, *cell_start;
};

// What the probe's continuous coordinates come out in: pixels, or (beta) theta_E,
// pixel coordinate u at x0 + u dx.
struct LmUnits {
    double x0 = 0, y0 = 0, dx = 1, dy = 1;
    bool beta = false;
    LmUnits() = default;
    LmUnits(double x0_, double y0_, double dx_, double dy_, bool b)
        : x0(x0_), y0(y0_), dx(dx_), dy(dy_), beta(b)
    {
    }
};

// Short lists passed by value: light-curve rows, and the first pixel column of
// each bin and the end of the last.
#define LM_ARG_TRACKS 64
#define LM_ARG_BINS 511
struct LmTracks {
    int32_t row[LM_ARG_TRACKS];
};
struct LmBins {
    int32_t col[LM_ARG_BINS + 1];
};

// Launchers implemented in lm_kernels.hip (return hipError_t as int).
// Lens arrays from a pinned block: n x, y, m (doubles), n I and J, nstart CSR entries.
int lm_launch_lens_upload(const double* src, int64_t n, int64_t nstart, const LmLensArrays& o,
                          void* stream);
// The precision probe: n lattice rays (every ray when n is the lattice's number), and
// part[3 k] .. = sums of the moves of a and c against b and the rays in the map, per workgroup.
int lm_launch_probe_rays(int64_t nx, int64_t ny, int64_t n, int64_t* ii, int64_t* jj,
                         void* stream);
int lm_launch_probe_moves(const double* a, const double* c, const double* b, int64_t n, int snx,
                          int sny, double* part, int parts, void* stream);
// The rectangle sheet's holomorphic part added to every level-2 cell's
// coefficients (after the far-field kernels).
int lm_launch_sheet(const LmDesc& d, int terms, LmCoef* coef, void* stream);
int lm_launch_coeffs(const LmDesc& d, int precision, int terms, int64_t ci0, int64_t cj0,
                     int64_t nci, int64_t ncj, LmCoef* out, void* stream);
// Hierarchical far field: level-1 series (d.Q terms) into d.l1exp, then the
// coefficients of every level-2 cell.
int lm_launch_coeffs_hier(const LmDesc& d, int terms, LmCoef* out, void* stream);
// Near-lens deflection of every level-2 cell centre (LmCoef::n0x, n0y) for the
// centred near sums; the rest of each record is left as it is.
int lm_launch_near_centre(const LmDesc& d, LmCoef* out, void* stream);
int lm_launch_shoot_map(const LmDesc& d, int scheme, int precision, int terms, int rays_per_lane,
                        void* stream);
// layout: an LDS layout (above); LM_LAYOUTS pairs it is not built for give
// hipErrorInvalidValue
int lm_launch_shoot_batch(const LmDesc* descs, const int64_t* offsets, const int32_t* order,
                          int nmaps, unsigned long long* queue, int scheme, int precision,
                          int terms, int rays_per_lane, int layout, int grid, void* stream);
int lm_launch_fill_u64(unsigned long long* p, int64_t n, unsigned long long v, void* stream);
int lm_launch_reset_counts(unsigned long long* counts, int64_t n, unsigned long long* n_out,
                           void* stream);
// Entries [first, first + n) of a window of the map (np columns from (p0, q0);
// whole: the map) to pinned host memory, as counts or (mu) counts x factor, and
// *extra (may be null) after them.
int lm_launch_read_back(const unsigned long long* map, int64_t snx, int64_t p0, int64_t q0,
                        int64_t np, bool whole, bool mu, int64_t first, int64_t n, double factor,
                        unsigned long long* out, const unsigned long long* extra, void* stream);
// part[0..parts) = partial sums of p[0..n)
int lm_launch_sum_u64(const unsigned long long* p, int64_t n, unsigned long long* part, int parts,
                      void* stream);
// p, q: pixels (-1 outside the map; may be null); uv (may be null): continuous pixel
// coordinates, 2 per ray, that the pixels are the floor of
int lm_launch_trace(const LmDesc& d, int scheme, int precision, int terms, const int64_t* ii,
                    const int64_t* jj, int64_t n, int32_t* p, int32_t* q, double* uv,
                    const LmUnits& units, void* stream);
int lm_launch_deflect(const LmDesc& d, int scheme, int precision, int terms, const double* th,
                      int64_t n, double* alpha, void* stream);
// Rows from `tracks`, or from `rows` where it is null (nt <= LM_ARG_TRACKS).
int lm_launch_peaks(const unsigned long long* counts, int64_t nx, int64_t ny, const LmTracks& rows,
                    const int32_t* tracks, int64_t nt, int k, uint8_t* flags, void* stream);
// out[b], out[nb + b] = true peaks of the listed rows in the columns [col[b],
// col[b+1]) and the sum of their counts; col from `cols`, or from `bins` where it
// is null (nb <= LM_ARG_BINS); c0 = col[0], c1 = col[nb].  hist (2 nb) and *done
// are zero before and after.
int lm_launch_peak_stats(const unsigned long long* counts, int64_t nx, int64_t ny,
                         const LmTracks& rows, const int32_t* tracks, int64_t nt, int k,
                         const LmBins& bins, const int32_t* cols, int c0, int c1, int nb,
                         unsigned long long* hist, unsigned* done, unsigned long long* out,
                         void* stream);
// n indices from pinned to device memory
int lm_launch_copy_i32(const int32_t* src, int64_t n, int32_t* dst, void* stream);
int lm_shoot_occupancy(int scheme, int precision, int terms, int rays_per_lane, int layout,
                       int* wg_per_cu);
// Device address of the current device's scratch array (resolved once per
// device); returns a hipError_t.
int lm_scratch_address(void** out);
bool lm_supported_rays_per_lane(int r);

// Per-pair instances of the shooting kernels, probes and their launchers
// (lm_shoot_inst.hip, compiled once per (scheme, precision) pair).
#define LM_INST_CAT2(base, s, p) base##_s##s##_p##p
#define LM_INST_CAT(base, s, p) LM_INST_CAT2(base, s, p)
#define LM_INST_DECLARE(S, PR)                                                                \
    int LM_INST_CAT(lm_inst_shoot_map, S, PR)(const LmDesc& d, int nr, int terms, void* stream); \
    int LM_INST_CAT(lm_inst_shoot_batch, S, PR)(const LmDesc* descs, const int64_t* offs,     \
                                                const int32_t* order, int nmaps,              \
                                                unsigned long long* queue, int nr, int terms, \
                                                int layout, int grid, void* stream);          \
    int LM_INST_CAT(lm_inst_occupancy, S, PR)(int nr, int terms, int layout, int* wg_per_cu); \
    int LM_INST_CAT(lm_inst_trace, S, PR)(const LmDesc& d, int terms, const int64_t* ii,      \
                                          const int64_t* jj, int64_t n, int32_t* p,           \
                                          int32_t* q, double* uv, const LmUnits& units,       \
                                          void* stream);                                      \
    int LM_INST_CAT(lm_inst_deflect, S, PR)(const LmDesc& d, int terms, const double* th,     \
                                            int64_t n, double* alpha, void* stream);
LM_INST_DECLARE(0, 0)
LM_INST_DECLARE(0, 1)
LM_INST_DECLARE(1, 0)
LM_INST_DECLARE(1, 1)
LM_INST_DECLARE(1, 2)
LM_INST_DECLARE(1, 4)
