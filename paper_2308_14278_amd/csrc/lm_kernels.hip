// lm_kernels.hip -- gfx950 kernels of liblensmap besides the shooting kernels
// (lm_device.h, instantiated per scheme and precision in lm_shoot_inst.hip),
// and the entry points that launch every kernel.
//
//  k_coeffs       far-field Taylor coefficients of every level-2 cell (Sec. 3.2.2):
//                 a_n = -sum_{far k} m_k / (z_k - z_c)^(n+1); ranges of far
//                 lenses read through the scalar cache, FP64 arithmetic.
//  k_l1_expand    hierarchical far field (optional): series per level-1 cell,
//  k_l1_shift     re-expanded about every level-2 centre.
//  k_sum_u64, k_fill_u64, k_reset_counts   reductions and fills of count buffers.
//
// The shooting kernels (k_shoot_map: one workgroup per tile of level-2 cells;
// k_shoot_batch: persistent, tiles of many maps from a queue) sum the near
// lenses directly (Eq. 9) on offsets rebased to the cell centre (FP32, or FP64
// in the FP64 near-sum mode), add the far-field Taylor series and the macro
// map with the sheet term (Eq. 6) re-expanded per ray row, bin in FP64 pixel
// coordinates, and count (Sec. 3.2.3) through per-lane runs, a wave merge and
// an LDS window flushed to the uint64 map.
#include "lm_device.h"

namespace {

// One far-field term added to a cell's coefficients: with w = z_k - z_c, u =
// 1 / w = conj(w) / |w|^2 and t = m u^(n+1), a_n -= t.
template <int P, class T>
__device__ __forceinline__ void coef_term(T wx, T wy, T m, T tiny, T* ar, T* ai)
{
    const T r2 = fma(wx, wx, fma(wy, wy, tiny));
    const T inv = recip_nr2(r2);
    const T ux = wx * inv, uy = -wy * inv;
    T tx = m * ux, ty = m * uy;
#pragma unroll
    for (int n = 0; n < P; ++n) {
        ar[n] -= tx;
        ai[n] -= ty;
        if (n + 1 < P) {
            const T nx = fma(tx, ux, -(ty * uy));
            const T ny = fma(tx, uy, ty * ux);
            tx = nx;
            ty = ny;
        }
    }
}

// Far-field coefficients: one level-2 cell per lane, every lens in list order.
// Bound: FP64 issue (33 FP64 instructions a lens and cell).  The lenses are
// sorted by level-1 cell, so those near some cell of the wave -- the level-1
// cells within H of the wave's -- are one range per level-1 row; the lenses
// between the ranges are far for every lane and need no test, and those inside
// are tested lane by lane.  A lens is the same for the whole wave: its data come
// through the scalar cache, four lenses to a load and one load ahead, since the few
// waves of a lattice of few cells have nothing else to hide it behind.  The whole call
// (us; every lens staged in LDS and tested / read as it is summed / one load ahead):
//   13000 lenses, 2.9e6 cells         44700  41050  38890
//   13000 lenses, lattice of 1e6 rays  2308   3020   1929
//   13000 lenses, lattice of 1e5 rays  3559   5055   3377
template <int PREC, int P>
__global__ __launch_bounds__(kWG) void k_coeffs(LmDesc d, int64_t ci0, int64_t cj0, int64_t nci,
                                                int64_t ncj, LmCoef* __restrict__ out)
{
    typedef typename std::conditional<PREC != 1, double, float>::type T;
    const int64_t c = (int64_t)blockIdx.x * kWG + threadIdx.x, nc = nci * ncj;
    const bool valid = c < nc;
    const int64_t ci = ci0 + (valid ? c % nci : 0), cj = cj0 + (valid ? c / nci : 0);
    const int I = (int)(ci / d.Kx), J = (int)(cj / d.Ky);
    // near: |I_k - I| <= H and |J_k - J| <= H, as one unsigned range test per axis
    const int Ilo = I - d.H, Jlo = J - d.H;
    const unsigned span = 2u * (unsigned)d.H;
    // keeps r^2 of a lens at the cell centre (always near) away from zero; no
    // effect on any far lens
    const T tiny = PREC != 1 ? (T)1e-300 : (T)1e-30f;
    T zx, zy;
    if (PREC != 1) {
        zx = (T)cell_cx(d, ci);
        zy = (T)cell_cy(d, cj);
    } else {
        zx = (T)cell_cxf(d, ci);
        zy = (T)cell_cyf(d, cj);
    }
    T ar[P], ai[P];
#pragma unroll
    for (int n = 0; n < P; ++n) {
        ar[n] = 0;
        ai[n] = 0;
    }
    ConstP<T> lx, ly, lm;
    if constexpr (PREC != 1) {
        lx = (ConstP<T>)d.lx;
        ly = (ConstP<T>)d.ly;
        lm = (ConstP<T>)d.lmd;
    } else {
        lx = (ConstP<T>)d.lxf;
        ly = (ConstP<T>)d.lyf;
        lm = (ConstP<T>)d.lmf;
    }
    ConstP<int32_t> lI = (ConstP<int32_t>)d.lI, lJ = (ConstP<int32_t>)d.lJ;
    // Lenses k .. e - 1, four at a time, the next four read while the current are summed.
    // TEST: those in a lane's near block add nothing.
    auto range = [&](auto test, int k, int e) __attribute__((always_inline)) {
        constexpr bool TEST = decltype(test)::value;
        constexpr int N = 4;
        struct Group {
            T x[N], y[N], m[N];
            int I[N], J[N];
        };
        auto load1 = [&](Group& g, int q, int i) __attribute__((always_inline)) {
            g.x[q] = lx[i];
            g.y[q] = ly[i];
            g.m[q] = lm[i];
            if constexpr (TEST) {
                g.I[q] = lI[i];
                g.J[q] = lJ[i];
            }
        };
        auto load = [&](Group& g, int i) __attribute__((always_inline)) {
            // Apart from the loads of the group before, and behind their arrival: scalar
            // loads come back in any order, so a wait for those would wait for these.
            asm volatile("" : "+s"(i));
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
#pragma unroll
            for (int q = 0; q < N; ++q) load1(g, q, i + q);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto add1 = [&](const Group& g, int q) __attribute__((always_inline)) {
            T m = g.m[q];
            if constexpr (TEST) {
                const bool near =
                    ((unsigned)(g.I[q] - Ilo) <= span) & ((unsigned)(g.J[q] - Jlo) <= span);
                m = near ? (T)0 : m;
            }
            coef_term<P>(g.x[q] - zx, g.y[q] - zy, m, tiny, ar, ai);
        };
        auto add = [&](const Group& g) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < N; ++q) add1(g, q);
        };
        Group g, h;
        if (k + N <= e) {
            load(g, k);
            for (; k + 3 * N <= e; k += 2 * N) {
                load(h, k + N);
                add(g);
                load(g, k + 2 * N);
                add(h);
            }
            if (k + 2 * N <= e) {
                load(h, k + N);
                add(g);
                g = h;
                k += N;
            }
            add(g);
            k += N;
        }
        if (k < e) {
#pragma unroll
            for (int q = 0; q < N - 1; ++q) load1(g, q, min(k + q, e - 1));
#pragma unroll
            for (int q = 0; q < N - 1; ++q)
                if (k + q < e) add1(g, q);
        }
    };
    auto far = [&](int k, int e) __attribute__((always_inline)) {
        range(std::false_type{}, k, e);
    };
    auto tested = [&](int k, int e) __attribute__((always_inline)) {
        range(std::true_type{}, k, e);
    };
    // the level-1 cells of the wave's cells c .. c + 63, one or more rows of them
    const int64_t w0 = c - (threadIdx.x & 63);
    const int n = (int)d.nlens;
    if (w0 < nc) {
        const int64_t w1 = min(w0 + 63, nc - 1);
        const int64_t r0 = w0 / nci, r1 = w1 / nci;
        const bool one = r0 == r1;  // cells of one row, else any column
        // (the same in every lane: scalars, as everything derived from them)
        auto uniform = [](int64_t v) { return __builtin_amdgcn_readfirstlane((int)v); };
        const int i0 = uniform((ci0 + (one ? w0 - r0 * nci : 0)) / d.Kx);
        const int i1 = uniform((ci0 + (one ? w1 - r0 * nci : nci - 1)) / d.Kx);
        const int j0 = uniform((cj0 + r0) / d.Ky), j1 = uniform((cj0 + r1) / d.Ky);
        ConstP<int32_t> cs = (ConstP<int32_t>)d.cell_start;
        int k = 0;
        // padded rows j0 - H .. j1 + H and columns i0 - H .. i1 + H
        for (int r = j0; r <= j1 + 2 * d.H; ++r) {
            const int s = cs[r * d.nl1x + i0], e = cs[r * d.nl1x + i1 + 2 * d.H + 1];
            far(k, s);
            tested(s, e);
            k = e;
        }
        far(k, n);
    }
    if (valid) {
        LmCoef& o = out[cj * d.ncx + ci];
        o.a0r = (double)ar[0];
        o.a0i = (double)ai[0];
#pragma unroll
        for (int n = 1; n < 7; ++n) {
            o.a[2 * (n - 1)] = n < P ? (float)ar[n < P ? n : 0] : 0.f;
            o.a[2 * (n - 1) + 1] = n < P ? (float)ai[n < P ? n : 0] : 0.f;
        }
    }
}

// Centre of box (sx, sy) of level-1 cell (I, J) of the hierarchical far
// field: the level-1 cell's centre when it is one box along that axis, else
// the centre of the box's level-2 cells (boxes of d.bx x d.by cells, the last
// one narrower).
__device__ __forceinline__ void box_centre(const LmDesc& d, int64_t I, int64_t J, int sx, int sy,
                                           double& Zx, double& Zy)
{
    if (d.nbx == 1) {
        Zx = d.x0 + ((double)I + 0.5) * (double)((int64_t)d.Kx * d.R) * d.dx;
    } else {
        const int64_t c0 = I * d.Kx + (int64_t)sx * d.bx;
        const int64_t c1 = min(c0 + d.bx, (I + 1) * d.Kx);
        Zx = d.x0 + 0.5 * (double)(c0 + c1) * (double)d.R * d.dx;
    }
    if (d.nby == 1) {
        Zy = d.y0 + ((double)J + 0.5) * (double)((int64_t)d.Ky * d.R) * d.dy;
    } else {
        const int64_t r0 = J * d.Ky + (int64_t)sy * d.by;
        const int64_t r1 = min(r0 + d.by, (J + 1) * d.Ky);
        Zy = d.y0 + 0.5 * (double)(r0 + r1) * (double)d.R * d.dy;
    }
}

// Threads of step 1 below: the Q terms are cut into ns = ceil(Q / 8) slices of
// eight, a box's lenses into ng = 256 / ns groups (group g holds every ng-th far
// lens), and a thread sums SL consecutive slices of a group's lenses: all of them
// up to five, else half, so that nsg threads share a group.
struct L1Split {
    int ns, ng, SL, nsg, boxes;
};

__host__ __device__ inline L1Split l1_split(int Q)
{
    L1Split f;
    f.ns = (Q + 7) >> 3;
    f.ng = kWG / f.ns;
    f.nsg = f.ns <= 5 ? 1 : 2;
    f.SL = (f.ns + f.nsg - 1) / f.nsg;
    f.boxes = kWG / (f.ng * f.nsg);
    return f;
}

// Hierarchical far field, step 1: the series of the far lenses of level-1 cell
// (I, J) about the centre Z of one of its boxes, A_n = -sum_far m_k / (z_k -
// Z)^(n+1), n < Q <= 64 (the level-2 series of Sec. 3.2.2 taken one level up).
// A workgroup takes as many boxes as its threads make (L1Split); then, box after
// box, threads n < Q add the groups' partial sums in a fixed order.
// Bound: FP64 issue.  A lens costs ~35 instructions for 1 / (z_k - Z) and its
// eighth power and ~64 for each slice, the first of them once per thread: with
// one slice per thread they were paid ns times (71115 boxes, 2749 lenses, Q = 24:
// 1.75 ms, 2.66 so).
template <int SL>
__global__ __launch_bounds__(kWG) void k_l1_expand(LmDesc d, int64_t nboxes)
{
    __shared__ double2 part[8 * kWG];  // [groups][8 ns] of one box
    const L1Split f = l1_split(d.Q);
    const int tid = threadIdx.x, per = f.ng * f.nsg;
    const int mine = tid / per, sg = (tid - mine * per) / f.ng, grp = tid % f.ng;
    const int64_t box0 = (int64_t)blockIdx.x * f.boxes;  // row-major over [n1y nby][n1x nbx]
    const int64_t cell = box0 + mine;
    const bool active = mine < f.boxes && cell < nboxes;
    const int s0 = sg * SL;
    double ar[8 * SL], ai[8 * SL];
#pragma unroll
    for (int j = 0; j < 8 * SL; ++j) {
        ar[j] = 0.0;
        ai[j] = 0.0;
    }
    if (active) {
        const int64_t bi = cell % (d.n1x * d.nbx), bj = cell / (d.n1x * d.nbx);
        const int64_t I = bi / d.nbx, J = bj / d.nby;
        double Zx, Zy;
        box_centre(d, I, J, (int)(bi % d.nbx), (int)(bj % d.nby), Zx, Zy);
        for (int64_t k = grp; k < d.nlens; k += f.ng) {
            if (abs(d.lI[k] - (int)I) <= d.H && abs(d.lJ[k] - (int)J) <= d.H) continue;
            const double wx = d.lx[k] - Zx, wy = d.ly[k] - Zy;
            const double iw2 = 1.0 / (wx * wx + wy * wy);
            const double ux = wx * iw2, uy = -wy * iw2;  // 1 / (z_k - Z)
            double px = ux, py = uy;  // u^8 by three squarings
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const double nx = px * px - py * py, ny = 2.0 * px * py;
                px = nx;
                py = ny;
            }
            // first term of slice s: m u^(8 s + 1)
            double bx = d.lmd[k] * ux, by = d.lmd[k] * uy;
            auto next_slice = [&] {
                const double nx = bx * px - by * py, ny = bx * py + by * px;
                bx = nx;
                by = ny;
            };
            for (int q = 0; q < s0; ++q) next_slice();
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                if (s > 0) next_slice();
                double tx = bx, ty = by;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    ar[8 * s + j] -= tx;
                    ai[8 * s + j] -= ty;
                    const double nx = tx * ux - ty * uy, ny = tx * uy + ty * ux;
                    tx = nx;
                    ty = ny;
                }
            }
        }
    }
    for (int b = 0; b < f.boxes && box0 + b < nboxes; ++b) {
        if (mine == b) {
            // term n of group g sits at 8 ns g + n
#pragma unroll
            for (int j = 0; j < 8 * SL; ++j)
                if (8 * s0 + j < 8 * f.ns)
                    part[8 * (f.ns * grp + s0) + j] = make_double2(ar[j], ai[j]);
        }
        __syncthreads();
        if (tid < d.Q) {
            double sr = 0.0, si = 0.0;
            for (int g = 0; g < f.ng; ++g) {
                sr += part[8 * f.ns * g + tid].x;
                si += part[8 * f.ns * g + tid].y;
            }
            d.l1exp[2 * ((box0 + b) * d.Q + tid)] = sr;
            d.l1exp[2 * ((box0 + b) * d.Q + tid) + 1] = si;
        }
        __syncthreads();
    }
}

// Hierarchical far field, step 2: the series of step 1 of the box holding each
// level-2 cell re-expanded about the cell's centre z_c, a_p = sum_{n>=p}
// C(n,p) A_n (z_c - Z)^(n-p), with T_n[p] = C(n,p) w^(n-p) advanced by
// T_{n+1}[p] = w T_n[p] + T_n[p-1].
template <int P>
__global__ __launch_bounds__(kWG) void k_l1_shift(LmDesc d, LmCoef* __restrict__ out)
{
    const int64_t c = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (c >= d.ncx * d.ncy) return;
    const int64_t ci = c % d.ncx, cj = c / d.ncx;
    const int64_t I = ci / d.Kx, J = cj / d.Ky;
    const int sx = (int)((ci - I * d.Kx) / d.bx), sy = (int)((cj - J * d.Ky) / d.by);
    double Zx, Zy;
    box_centre(d, I, J, sx, sy, Zx, Zy);
    const int64_t box = (J * d.nby + sy) * (d.n1x * d.nbx) + (I * d.nbx + sx);
    const double wx = cell_cx(d, ci) - Zx, wy = cell_cy(d, cj) - Zy;
    double tr[P], ti[P], ar[P], ai[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        tr[p] = p == 0 ? 1.0 : 0.0;
        ti[p] = 0.0;
        ar[p] = 0.0;
        ai[p] = 0.0;
    }
    const double* A = d.l1exp + 2 * (box * d.Q);
    for (int n = 0; n < d.Q; ++n) {
        const double Ar = A[2 * n], Ai = A[2 * n + 1];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            ar[p] += Ar * tr[p] - Ai * ti[p];
            ai[p] += Ar * ti[p] + Ai * tr[p];
        }
#pragma unroll
        for (int p = P - 1; p >= 0; --p) {
            const double nr = tr[p] * wx - ti[p] * wy + (p > 0 ? tr[p > 0 ? p - 1 : 0] : 0.0);
            const double ni = tr[p] * wy + ti[p] * wx + (p > 0 ? ti[p > 0 ? p - 1 : 0] : 0.0);
            tr[p] = nr;
            ti[p] = ni;
        }
    }
    LmCoef& o = out[cj * d.ncx + ci];
    o.a0r = ar[0];
    o.a0i = ai[0];
#pragma unroll
    for (int n = 1; n < 7; ++n) {
        o.a[2 * (n - 1)] = n < P ? (float)ar[n < P ? n : 0] : 0.f;
        o.a[2 * (n - 1) + 1] = n < P ? (float)ai[n < P ? n : 0] : 0.f;
    }
}

// Sum of p[0..n), one partial sum per workgroup.  Bound by HBM: 16-byte loads,
// four in flight per lane (2.15 GB in 0.94 ms with one 8-byte load at a time,
// 0.39 ms so).
__global__ __launch_bounds__(kWG) void k_sum_u64(const unsigned long long* __restrict__ p,
                                                 int64_t n, unsigned long long* __restrict__ part)
{
    __shared__ unsigned long long ws[LM_WAVES];
    const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x, nt = (int64_t)gridDim.x * kWG;
    unsigned long long s = 0;
    // the caller's buffer is aligned to 8 bytes: its first entry may stand alone
    const int64_t head = ((uintptr_t)p & 15) && n > 0 ? 1 : 0;
    const ulonglong2* v = (const ulonglong2*)(p + head);
    const int64_t nv = (n - head) >> 1;
    int64_t i = t;
    for (; i + 3 * nt < nv; i += 4 * nt) {
        const ulonglong2 a = v[i], b = v[i + nt], c = v[i + 2 * nt], e = v[i + 3 * nt];
        s += (a.x + a.y) + (b.x + b.y) + (c.x + c.y) + (e.x + e.y);
    }
    for (; i < nv; i += nt) s += v[i].x + v[i].y;
    if (t == 0) {
        if (head) s += p[0];
        if ((n - head) & 1) s += p[n - 1];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < LM_WAVES; ++w) s += ws[w];
        part[blockIdx.x] = s;
    }
}

__global__ void k_fill_u64(unsigned long long* p, int64_t n, unsigned long long v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// A map's counts and its count of rays outside, cleared in one launch: on a map
// of a few thousand pixels a launch takes longer than the writes, and a reset in
// two was a quarter of what a reset, a shot and a read of it submit.
__global__ void k_reset_counts(unsigned long long* counts, int64_t n, unsigned long long* n_out)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) *n_out = 0;
    for (int64_t i = t; i < n; i += (int64_t)gridDim.x * blockDim.x) counts[i] = 0;
}

// Entries [first, first + n) of a window of a row-major map of width snx -- rows
// from q0, np columns from p0, row after row (WHOLE: the map itself) -- written
// to pinned host memory: the counts, or (MU) the magnifications counts x factor,
// converted and rounded as the host would; and *extra after them, if given.
// Bound by the bus (57 GB/s): no device copy is made first and none of the
// conversion is left to the host.
template <bool WHOLE, bool MU>
__global__ __launch_bounds__(kWG) void k_read_back(const unsigned long long* __restrict__ map,
                                                   int64_t snx, int64_t p0, int64_t q0, int64_t np,
                                                   int64_t first, int64_t n, double factor,
                                                   unsigned long long* __restrict__ out,
                                                   const unsigned long long* __restrict__ extra)
{
    const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x;
    for (int64_t i = t; i < n; i += (int64_t)gridDim.x * kWG) {
        int64_t e = first + i;
        if (!WHOLE) {
            const int64_t r = e / np;
            e = (q0 + r) * snx + p0 + (e - r * np);
        }
        const unsigned long long c = map[e];
        out[i] = MU ? (unsigned long long)__double_as_longlong((double)c * factor) : c;
    }
    if (t == 0 && extra) out[n] = *extra;
}

// --------------------------------------------- a new lens field

// The lens arrays from one pinned block (n x, y, m as doubles, then n I and J,
// then nstart CSR entries): every array, the FP32 copies among them, in one
// launch, where nine copies from pageable memory took most of the call
// (latency: ~12 us each).
__global__ __launch_bounds__(kWG) void k_lens_upload(const double* __restrict__ src, int64_t n,
                                                     int64_t nstart, LmLensArrays o)
{
    const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x;
    const int32_t* cells = (const int32_t*)(src + 3 * n);
    if (t < n) {
        const double x = src[t], y = src[n + t], m = src[2 * n + t];
        o.lx[t] = x;
        o.ly[t] = y;
        o.lmd[t] = m;
        o.lxf[t] = (float)x;
        o.lyf[t] = (float)y;
        o.lmf[t] = (float)m;
        o.lI[t] = cells[t];
        o.lJ[t] = cells[n + t];
    }
    if (t < nstart) o.cell_start[t] = cells[2 * n + t];
}

__device__ __forceinline__ uint64_t splitmix64(uint64_t x)
{
    x += 0x9e3779b97f4a7c15ull;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

// The precision probe's rays: all n of a lattice of n rays, else n at fixed
// counter-based positions.
__global__ __launch_bounds__(kWG) void k_probe_rays(int64_t nx, int64_t ny, int64_t n, bool all,
                                                    int64_t* __restrict__ ii,
                                                    int64_t* __restrict__ jj)
{
    const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (t >= n) return;
    ii[t] = all ? t % nx : (int64_t)(splitmix64(2 * (uint64_t)t) % (uint64_t)nx);
    jj[t] = all ? t / nx : (int64_t)(splitmix64(2 * (uint64_t)t + 1) % (uint64_t)ny);
}

// How far plain (a) and centred (c) FP32 near sums move the images of the
// probe's rays from those with FP64 near sums (b): per workgroup the sums of
// |du| + |dv| (at most 1 a ray, 1 for a non-finite one) over the rays whose
// images lie in the map, and their number.
__global__ __launch_bounds__(kWG) void k_probe_moves(const double2* __restrict__ a,
                                                     const double2* __restrict__ c,
                                                     const double2* __restrict__ b, int64_t n,
                                                     double snx, double sny,
                                                     double* __restrict__ part)
{
    __shared__ double ws[3][LM_WAVES];
    double s[3] = {0.0, 0.0, 0.0};
    auto move = [](double du, double dv) {
        const double mv = fabs(du) + fabs(dv);
        return mv < 1.0 ? mv : 1.0;
    };
    for (int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * kWG) {
        const double2 v = b[t];
        if (!(v.x >= 0.0 && v.x < snx && v.y >= 0.0 && v.y < sny)) continue;
        const double2 p = a[t], q = c[t];
        s[0] += move(p.x - v.x, p.y - v.y);
        s[1] += move(q.x - v.x, q.y - v.y);
        s[2] += 1.0;
    }
    for (int k = 0; k < 3; ++k) {
        for (int o = 32; o > 0; o >>= 1) s[k] += __shfl_xor(s[k], o, 64);
        if ((threadIdx.x & 63) == 0) ws[k][threadIdx.x >> 6] = s[k];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double v = 0.0;
        for (int w = 0; w < LM_WAVES; ++w) v += ws[threadIdx.x][w];
        part[3 * blockIdx.x + threadIdx.x] = v;
    }
}

// ------------------------------------------------ the rectangle sheet

struct Cd {
    double r, i;
};
__device__ __forceinline__ Cd cd(double r, double i) { return Cd{r, i}; }
__device__ __forceinline__ Cd operator+(Cd a, Cd b) { return cd(a.r + b.r, a.i + b.i); }
__device__ __forceinline__ Cd operator-(Cd a, Cd b) { return cd(a.r - b.r, a.i - b.i); }
__device__ __forceinline__ Cd operator*(Cd a, Cd b)
{
    return cd(a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r);
}
__device__ __forceinline__ Cd operator*(double s, Cd a) { return cd(s * a.r, s * a.i); }
__device__ __forceinline__ Cd cinv(Cd a)
{
    const double n = a.r * a.r + a.i * a.i;
    return cd(a.r / n, -a.i / n);
}
// principal logarithm of wq / wp
__device__ __forceinline__ Cd clog_ratio(Cd wq, Cd wp)
{
    const double qr = wq.r * wp.r + wq.i * wp.i, qi = wq.i * wp.r - wq.r * wp.i;
    const double nq = wq.r * wq.r + wq.i * wq.i, np = wp.r * wp.r + wp.i * wp.i;
    return cd(0.5 * log(nq / np), atan2(qi, qr));
}

// The sheet of density -kappa_star on the lenses' rectangle (Sec. 2, Eq. 6):
// inside the rectangle its term in the lens equation is kappa_star theta +
// h(theta), and by Green's theorem on the rectangle
//   conj(h)(z) = (kappa_star / 2 pi i) oint z'* / (z - z') dz'
// over its edges, counter-clockwise.  About an expansion point z_e inside,
// conj(h) = sum_n H_n (z - z_e)^n with H_n = -(kappa_star / 2 pi i) J_n,
//   J_n = oint z'* w^-(n+1) dz',  w = z' - z_e.
// On an edge z'* is linear in z' (y = y_e: z'* = z' - 2 i y_e; x = x_e:
// z'* = 2 x_e - z'), so z'* = s w + c there and each edge from wP to wQ gives
//   n = 0:  s (wQ - wP) + c Log(wQ / wP)
//   n = 1:  s Log(wQ / wP) + c (1/wP - 1/wQ)
//   n >= 2: s (wQ^(1-n) - wP^(1-n)) / (1 - n) + c (wP^-n - wQ^-n) / n
// (a straight edge that misses z_e turns by less than pi about it, so the
// principal logarithm of the ratio is the integral).  The far field enters the
// lens equation as -alpha_far with conj(alpha_far) = sum a_n delta^n and the
// sheet as +h, so a_n gains -H_n = (kappa_star / 2 pi i) J_n.  z_e is the
// centre of the part of the cell inside the lattice (the cell centre except
// in a partial last column or row), and the polynomial is re-expanded about
// the cell centre: b'_k = sum_{n>=k} C(n,k) b_n t^(n-k), t = z_c - z_e.
template <int P>
__global__ __launch_bounds__(kWG) void k_sheet(LmDesc d, LmCoef* __restrict__ out)
{
    const int64_t c = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (c >= d.ncx * d.ncy) return;
    const int64_t ci = c % d.ncx, cj = c / d.ncx;
    const int64_t i1 = min((ci + 1) * (int64_t)d.R, d.nx), j1 = min((cj + 1) * (int64_t)d.R, d.ny);
    const Cd ze = cd(d.x0 + 0.5 * ((double)(ci * d.R) + (double)i1) * d.dx,
                     d.y0 + 0.5 * ((double)(cj * d.R) + (double)j1) * d.dy);
    const Cd corner[4] = {cd(d.sx0, d.sy0), cd(d.sx1, d.sy0), cd(d.sx1, d.sy1),
                          cd(d.sx0, d.sy1)};
    // z'* = s w + c on the four edges, counter-clockwise from (sx0, sy0)
    const double es[4] = {1.0, -1.0, 1.0, -1.0};
    const Cd ec[4] = {ze - cd(0.0, 2.0 * d.sy0), cd(2.0 * d.sx1, 0.0) - ze,
                      ze - cd(0.0, 2.0 * d.sy1), cd(2.0 * d.sx0, 0.0) - ze};
    Cd J[P];
#pragma unroll
    for (int n = 0; n < P; ++n) J[n] = cd(0.0, 0.0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const Cd wp = corner[e] - ze, wq = corner[(e + 1) & 3] - ze;
        const double s = es[e];
        const Cd cc = ec[e];
        const Cd L = clog_ratio(wq, wp);
        const Cd ip = cinv(wp), iq = cinv(wq);
        J[0] = J[0] + s * (wq - wp) + cc * L;
        if constexpr (P > 1) J[1] = J[1] + s * L + cc * (ip - iq);
        // wP^-(n-1), wQ^-(n-1) and wP^-n, wQ^-n, advanced by one power per n
        Cd pp = ip, pq = iq, p2 = ip * ip, q2 = iq * iq;
#pragma unroll
        for (int n = 2; n < P; ++n) {
            J[n] = J[n] + (s / (1.0 - n)) * (pq - pp) + (1.0 / n) * (cc * (p2 - q2));
            pp = p2;
            pq = q2;
            p2 = p2 * ip;
            q2 = q2 * iq;
        }
    }
    // b_n = (kappa_star / 2 pi i) J_n = (kappa_star / 2 pi) (Im J_n, -Re J_n)
    const double f = d.kappa_star / (2.0 * 3.14159265358979323846);
    Cd b[P];
#pragma unroll
    for (int n = 0; n < P; ++n) b[n] = cd(f * J[n].i, -f * J[n].r);
    const Cd t = cd(cell_cx(d, ci), cell_cy(d, cj)) - ze;
    LmCoef& o = out[cj * d.ncx + ci];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        Cd acc = cd(0.0, 0.0), tp = cd(1.0, 0.0);
        double binom = 1.0;
#pragma unroll
        for (int n = k; n < P; ++n) {
            acc = acc + binom * (b[n] * tp);
            tp = tp * t;
            binom = binom * (double)(n + 1) / (double)(n + 1 - k);
        }
        if (k == 0) {
            o.a0r += acc.r;
            o.a0i += acc.i;
        } else {
            o.a[2 * k - 2] = (float)((double)o.a[2 * k - 2] + acc.r);
            o.a[2 * k - 1] = (float)((double)o.a[2 * k - 1] + acc.i);
        }
    }
}

// Near-lens deflection of each level-2 cell centre, one cell per thread: the
// sum over the cell's near list, in list order, of m (z_c - z_k) / |z_c - z_k|^2
// in FP64 (the centred near sums add each ray's FP32 change from it).  NaN when
// a near lens lies within twice the cell's half-diagonal of the centre: there
// the change is not small, and the shooting kernel sums that cell's near
// lenses plainly.
__global__ __launch_bounds__(kWG) void k_near_centre(LmDesc d, LmCoef* __restrict__ out)
{
    const int64_t c = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (c >= d.ncx * d.ncy) return;
    const int64_t ci = c % d.ncx, cj = c / d.ncx;
    const double zcx = cell_cx(d, ci), zcy = cell_cy(d, cj);
    const double rc2 = (double)d.R * d.R * (d.dx * d.dx + d.dy * d.dy);
    const L1Cell l1 = l1_of(d, ci, cj);
    double sx = 0.0, sy = 0.0;
    bool close = false;
    for (int r = 0; r <= 2 * d.H; ++r) {
        int s, e;
        near_row(d, l1, r, s, e);
        for (int k = s; k < e; ++k) {
            const double ox = d.lx[k] - zcx, oy = d.ly[k] - zcy;
            const double r2 = ox * ox + oy * oy;
            close |= r2 < rc2;
            const double q = d.lmd[k] / r2;
            sx -= q * ox;
            sy -= q * oy;
        }
    }
    LmCoef& o = out[cj * d.ncx + ci];
    o.n0x = close ? __builtin_nan("") : sx;
    o.n0y = close ? __builtin_nan("") : sy;
}

}  // namespace

// Every (scheme, precision) pair lm_shoot_inst.hip is built for.
#define LM_PAIRS(X) X(0, 0) X(0, 1) X(1, 0) X(1, 1) X(1, 2) X(1, 4)

bool lm_supported_rays_per_lane(int r) { return r == 4 || r == 8 || r == 16; }

int lm_launch_shoot_map(const LmDesc& d, int scheme, int precision, int terms, int rays_per_lane,
                        void* stream)
{
    if (d.ntiles <= 0) return 0;
    if (scheme == 0 && terms != lm_direct_terms(d.nlens)) return (int)hipErrorInvalidValue;
#define X(S, PR)                                                                            \
    if (scheme == S && precision == PR)                                                     \
        return LM_INST_CAT(lm_inst_shoot_map, S, PR)(d, rays_per_lane, terms, stream);
    LM_PAIRS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int lm_launch_shoot_batch(const LmDesc* descs, const int64_t* offsets, const int32_t* order,
                          int nmaps, unsigned long long* queue, int scheme, int precision,
                          int terms, int rays_per_lane, int layout, int grid, void* stream)
{
#define X(S, PR)                                                                            \
    if (scheme == S && precision == PR)                                                     \
        return LM_INST_CAT(lm_inst_shoot_batch, S, PR)(descs, offsets, order, nmaps, queue, \
                                                       rays_per_lane, terms, layout, grid,  \
                                                       stream);
    LM_PAIRS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int lm_shoot_occupancy(int scheme, int precision, int terms, int rays_per_lane, int layout,
                       int* wg_per_cu)
{
#define X(S, PR)                                                                            \
    if (scheme == S && precision == PR)                                                     \
        return LM_INST_CAT(lm_inst_occupancy, S, PR)(rays_per_lane, terms, layout, wg_per_cu);
    LM_PAIRS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int lm_launch_trace(const LmDesc& d, int scheme, int precision, int terms, const int64_t* ii,
                    const int64_t* jj, int64_t n, int32_t* p, int32_t* q, double* uv,
                    const LmUnits& units, void* stream)
{
    if (n <= 0) return 0;
#define X(S, PR)                                                                            \
    if (scheme == S && precision == PR)                                                     \
        return LM_INST_CAT(lm_inst_trace, S, PR)(d, terms, ii, jj, n, p, q, uv, units, \
                                                 stream);
    LM_PAIRS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int lm_launch_deflect(const LmDesc& d, int scheme, int precision, int terms, const double* th,
                      int64_t n, double* alpha, void* stream)
{
    if (n <= 0) return 0;
#define X(S, PR)                                                                            \
    if (scheme == S && precision == PR)                                                     \
        return LM_INST_CAT(lm_inst_deflect, S, PR)(d, terms, th, n, alpha, stream);
    LM_PAIRS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int lm_launch_coeffs_hier(const LmDesc& d, int terms, LmCoef* out, void* stream)
{
    const int64_t n1 = d.n1x * d.nbx * d.n1y * d.nby, n2 = d.ncx * d.ncy;
    if (n1 <= 0 || n2 <= 0) return 0;
    if (d.Q < terms || d.Q > 64) return (int)hipErrorInvalidValue;
    hipStream_t s = (hipStream_t)stream;
    const L1Split f = l1_split(d.Q);
    const dim3 grid1((unsigned)((n1 + f.boxes - 1) / f.boxes));
    switch (f.SL) {
    case 1: hipLaunchKernelGGL(k_l1_expand<1>, grid1, dim3(kWG), 0, s, d, n1); break;
    case 2: hipLaunchKernelGGL(k_l1_expand<2>, grid1, dim3(kWG), 0, s, d, n1); break;
    case 3: hipLaunchKernelGGL(k_l1_expand<3>, grid1, dim3(kWG), 0, s, d, n1); break;
    case 4: hipLaunchKernelGGL(k_l1_expand<4>, grid1, dim3(kWG), 0, s, d, n1); break;
    default: hipLaunchKernelGGL(k_l1_expand<5>, grid1, dim3(kWG), 0, s, d, n1); break;
    }
    const int e = (int)hipGetLastError();
    if (e) return e;
    const dim3 grid((unsigned)((n2 + kWG - 1) / kWG));
    switch (terms) {
    case 1: hipLaunchKernelGGL(k_l1_shift<1>, grid, dim3(kWG), 0, s, d, out); break;
    case 2: hipLaunchKernelGGL(k_l1_shift<2>, grid, dim3(kWG), 0, s, d, out); break;
    case 3: hipLaunchKernelGGL(k_l1_shift<3>, grid, dim3(kWG), 0, s, d, out); break;
    case 4: hipLaunchKernelGGL(k_l1_shift<4>, grid, dim3(kWG), 0, s, d, out); break;
    case 5: hipLaunchKernelGGL(k_l1_shift<5>, grid, dim3(kWG), 0, s, d, out); break;
    case 6: hipLaunchKernelGGL(k_l1_shift<6>, grid, dim3(kWG), 0, s, d, out); break;
    case 7: hipLaunchKernelGGL(k_l1_shift<7>, grid, dim3(kWG), 0, s, d, out); break;
    default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

int lm_launch_sheet(const LmDesc& d, int terms, LmCoef* coef, void* stream)
{
    const int64_t n = d.ncx * d.ncy;
    if (n <= 0 || !d.sheet) return 0;
    const dim3 grid((unsigned)((n + kWG - 1) / kWG));
    hipStream_t s = (hipStream_t)stream;
    switch (terms) {
    case 1: hipLaunchKernelGGL(k_sheet<1>, grid, dim3(kWG), 0, s, d, coef); break;
    case 2: hipLaunchKernelGGL(k_sheet<2>, grid, dim3(kWG), 0, s, d, coef); break;
    case 3: hipLaunchKernelGGL(k_sheet<3>, grid, dim3(kWG), 0, s, d, coef); break;
    case 4: hipLaunchKernelGGL(k_sheet<4>, grid, dim3(kWG), 0, s, d, coef); break;
    case 5: hipLaunchKernelGGL(k_sheet<5>, grid, dim3(kWG), 0, s, d, coef); break;
    case 6: hipLaunchKernelGGL(k_sheet<6>, grid, dim3(kWG), 0, s, d, coef); break;
    case 7: hipLaunchKernelGGL(k_sheet<7>, grid, dim3(kWG), 0, s, d, coef); break;
    default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

int lm_launch_near_centre(const LmDesc& d, LmCoef* out, void* stream)
{
    const int64_t n = d.ncx * d.ncy;
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_near_centre, dim3((unsigned)((n + kWG - 1) / kWG)), dim3(kWG), 0,
                       (hipStream_t)stream, d, out);
    return (int)hipGetLastError();
}

int lm_launch_sum_u64(const unsigned long long* p, int64_t n, unsigned long long* part, int parts,
                      void* stream)
{
    if (parts <= 0) return 0;
    hipLaunchKernelGGL(k_sum_u64, dim3((unsigned)parts), dim3(kWG), 0, (hipStream_t)stream, p, n,
                       part);
    return (int)hipGetLastError();
}

int lm_launch_fill_u64(unsigned long long* p, int64_t n, unsigned long long v, void* stream)
{
    if (n <= 0) return 0;
    int64_t blocks = (n + kWG - 1) / kWG;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)blocks), dim3(kWG), 0, (hipStream_t)stream, p, n,
                       v);
    return (int)hipGetLastError();
}

int lm_launch_reset_counts(unsigned long long* counts, int64_t n, unsigned long long* n_out,
                           void* stream)
{
    int64_t blocks = (n + kWG - 1) / kWG;
    blocks = blocks < 1 ? 1 : blocks > 8192 ? 8192 : blocks;
    hipLaunchKernelGGL(k_reset_counts, dim3((unsigned)blocks), dim3(kWG), 0, (hipStream_t)stream,
                       counts, n, n_out);
    return (int)hipGetLastError();
}

int lm_launch_read_back(const unsigned long long* map, int64_t snx, int64_t p0, int64_t q0,
                        int64_t np, bool whole, bool mu, int64_t first, int64_t n, double factor,
                        unsigned long long* out, const unsigned long long* extra, void* stream)
{
    // a megabyte goes out in 512 workgroups of one entry per lane
    int64_t blocks = (n + kWG - 1) / kWG;
    blocks = blocks < 1 ? 1 : blocks > 512 ? 512 : blocks;
    const dim3 grid((unsigned)blocks);
    hipStream_t s = (hipStream_t)stream;
#define X(W, M)                                                                              \
    hipLaunchKernelGGL((k_read_back<W, M>), grid, dim3(kWG), 0, s, map, snx, p0, q0, np, first, n, \
                       factor, out, extra)
    if (whole && mu)
        X(true, true);
    else if (whole)
        X(true, false);
    else if (mu)
        X(false, true);
    else
        X(false, false);
#undef X
    return (int)hipGetLastError();
}

int lm_launch_lens_upload(const double* src, int64_t n, int64_t nstart, const LmLensArrays& o,
                          void* stream)
{
    const int64_t m = n > nstart ? n : nstart;
    if (m <= 0) return 0;
    hipLaunchKernelGGL(k_lens_upload, dim3((unsigned)((m + kWG - 1) / kWG)), dim3(kWG), 0,
                       (hipStream_t)stream, src, n, nstart, o);
    return (int)hipGetLastError();
}

int lm_launch_probe_rays(int64_t nx, int64_t ny, int64_t n, int64_t* ii, int64_t* jj,
                         void* stream)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_probe_rays, dim3((unsigned)((n + kWG - 1) / kWG)), dim3(kWG), 0,
                       (hipStream_t)stream, nx, ny, n, n == nx * ny, ii, jj);
    return (int)hipGetLastError();
}

int lm_launch_probe_moves(const double* a, const double* c, const double* b, int64_t n, int snx,
                          int sny, double* part, int parts, void* stream)
{
    hipLaunchKernelGGL(k_probe_moves, dim3((unsigned)parts), dim3(kWG), 0, (hipStream_t)stream,
                       (const double2*)a, (const double2*)c, (const double2*)b, n, (double)snx,
                       (double)sny, part);
    return (int)hipGetLastError();
}

int lm_launch_coeffs(const LmDesc& d, int precision, int terms, int64_t ci0, int64_t cj0,
                     int64_t nci, int64_t ncj, LmCoef* out, void* stream)
{
    const int64_t n = nci * ncj;
    if (n <= 0) return 0;
    const dim3 grid((unsigned)((n + kWG - 1) / kWG));
    hipStream_t s = (hipStream_t)stream;
#define LM_COEF(PR, P) \
    hipLaunchKernelGGL((k_coeffs<PR, P>), grid, dim3(kWG), 0, s, d, ci0, cj0, nci, ncj, out)
#define LM_COEF_P(PR)                         \
    switch (terms) {                          \
    case 1: LM_COEF(PR, 1); break;            \
    case 2: LM_COEF(PR, 2); break;            \
    case 3: LM_COEF(PR, 3); break;            \
    case 4: LM_COEF(PR, 4); break;            \
    case 5: LM_COEF(PR, 5); break;            \
    case 6: LM_COEF(PR, 6); break;            \
    case 7: LM_COEF(PR, 7); break;            \
    default: return (int)hipErrorInvalidValue; \
    }
    if (precision != 1) {
        LM_COEF_P(0)
    } else {
        LM_COEF_P(1)
    }
#undef LM_COEF_P
#undef LM_COEF
    return (int)hipGetLastError();
}
