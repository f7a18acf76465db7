// HIP kernels of the TDGL + Poisson time step (gfx950, wave64).
//
// Layout: fields are z-major with x fastest.  Multigrid levels with even x
// and y extents store their cells split by red/black colour (LevelArgs), so a
// Gauss-Seidel half-sweep streams contiguous arrays.  Workgroups are 64x4
// threads (one wave per row).  Every launch covers all instances of a batch:
// a block's global tile index is first remapped so that each of the 8 XCDs
// walks one contiguous range of tiles (consecutive planes and rows, keeping
// stencil neighbours in that XCD's L2), then split into (instance, tile) by a
// binary search in the launch's prefix table.
#include "fx_internal.h"

#include <hip/hip_ext.h>

namespace fx {

namespace {

__device__ __forceinline__ int wrap_p(int i, int n) { return i + 1 == n ? 0 : i + 1; }
__device__ __forceinline__ int wrap_m(int i, int n) { return i == 0 ? n - 1 : i - 1; }

// Explicit address spaces.  Pointers read from the instance table are
// generic; used as such they become flat instructions, which need 64-bit
// per-lane addresses and make every wait for a scalar load also wait for the
// vector loads in flight.  The kernels therefore view the arrays through
// global (1) pointers, and the coarse kernel its LDS copies through LDS (3)
// pointers.
#define FX_AS(n) __attribute__((address_space(n)))
template <int AS, typename T>
__device__ __forceinline__ T FX_AS(AS) *asp(T *p) { return (T FX_AS(AS) *)p; }

typedef InstState FX_AS(1) GState;
typedef double dpair __attribute__((ext_vector_type(2)));   // a 16-byte phi pair

template <typename T, int AS>
struct Lv {
    using value_type = T;
    int nx, ny, nz, rb;
    const T FX_AS(AS) *cxy, *czm, *czp, *dg;
    T FX_AS(AS) *e, *r, *sig;
    int sig_lo, sig_hi;
};

template <typename T, int AS = 1>
struct Xv {
    const int FX_AS(AS) *cks, *ccnt, *fthick, *cthick, *pka, *pkb;
    const T FX_AS(AS) *pwa, *pwb;
    int xy;
};

template <typename T>
__device__ __forceinline__ Lv<T, 1> gview(const LevelArgs<T> &L) {
    Lv<T, 1> v;
    v.nx = L.nx; v.ny = L.ny; v.nz = L.nz; v.rb = L.rb;
    v.cxy = asp<1>(L.cxy); v.czm = asp<1>(L.czm); v.czp = asp<1>(L.czp); v.dg = asp<1>(L.dg);
    v.e = asp<1>(L.e); v.r = asp<1>(L.r); v.sig = asp<1>(L.sig);
    v.sig_lo = L.sig_lo; v.sig_hi = L.sig_hi;
    return v;
}

template <typename T>
__device__ __forceinline__ Xv<T> xview(const XferArgs<T> &X) {
    Xv<T> v;
    v.cks = asp<1>(X.cks); v.ccnt = asp<1>(X.ccnt); v.fthick = asp<1>(X.fthick); v.cthick = asp<1>(X.cthick);
    v.pka = asp<1>(X.pka); v.pkb = asp<1>(X.pkb); v.pwa = asp<1>(X.pwa); v.pwb = asp<1>(X.pwb);
    v.xy = X.xy;
    return v;
}

// State of instance inst of a work-table launch, addressed from the kernel argument
// (one load, not a load of the pointer held in the instance and then of the state).
__device__ __forceinline__ GState *wstate(const Work &w, int inst) { return asp<1>(w.st + inst); }

struct Blk {
    int inst, t;
    bool ok;
};

__device__ __forceinline__ Blk find_block(const Work &w, int b, int nb) {
    const int g = (b & 7) * (nb >> 3) + (b >> 3);
    Blk r;
    r.ok = g < w.total;
    r.inst = 0;
    r.t = 0;
    if (!r.ok) return r;
    if (w.ninst == 1) {                       // prefix[0] = 0: no table lookup
        r.t = g;
        return r;
    }
    const int FX_AS(1) *pre = asp<1>(w.prefix);
    int lo = 0, hi = w.ninst;                 // largest lo with prefix[lo] <= g
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pre[mid] <= g) lo = mid;
        else hi = mid;
    }
    r.inst = __builtin_amdgcn_readfirstlane(lo);
    r.t = g - pre[r.inst];
    return r;
}
__device__ __forceinline__ Blk find_block(const Work &w) { return find_block(w, blockIdx.x, gridDim.x); }

struct T3 {
    int tx, ty, tz;
};
__device__ __forceinline__ T3 split3(int t, int nxw, int ny) {
    const int ntx = (nxw + BX - 1) / BX, nty = (ny + BY - 1) / BY;
    T3 r;
    r.tx = t % ntx;
    const int q = t / ntx;
    r.ty = q % nty;
    r.tz = q / nty;
    return r;
}

// The same tiles in z-fastest order (nzt tiles per column): consecutive tiles of one
// column share their halo planes, which the next tile then finds in L2.
__device__ __forceinline__ T3 split3z(int t, int nxw, int nzt) {
    const int ntx = (nxw + BX - 1) / BX;
    T3 r;
    r.tz = t % nzt;
    const int q = t / nzt;
    r.tx = q % ntx;
    r.ty = q / ntx;
    return r;
}

// Tile of 2^lbx x 2^(8-lbx) threads (a 256-thread block, x fastest); the
// smoother's tile shape is chosen per level at run time.
__device__ __forceinline__ T3 split3r(int t, int nxw, int ny, int lbx) {
    const int ntx = (nxw + (1 << lbx) - 1) >> lbx, nty = (ny + (256 >> lbx) - 1) >> (8 - lbx);
    T3 r;
    r.tx = t % ntx;
    const int q = t / ntx;
    r.ty = q % nty;
    r.tz = q / nty;
    return r;
}

dim3 grid_of(int total) { return dim3((total + 7) / 8 * 8); }

template <typename V>
__device__ __forceinline__ int cidx(const V &L, int i, int j, int k) {
    const int lin = (k * L.ny + j) * L.nx + i;
    if (!L.rb) return lin;
    return (((i + j + k) & 1) ? ((L.nx * L.ny * L.nz) >> 1) : 0) + (lin >> 1);
}

template <typename V>
__device__ __forceinline__ bool has_sig(const V &L, int k) { return k >= L.sig_lo && k < L.sig_hi; }

template <typename V>
__device__ __forceinline__ int sidx(const V &L, int i, int j, int k) {
    const int lin = ((k - L.sig_lo) * L.ny + j) * L.nx + i;
    if (!L.rb) return lin;
    return (((i + j + k) & 1) ? ((L.nx * L.ny * (L.sig_hi - L.sig_lo)) >> 1) : 0) + (lin >> 1);
}

// sum over the 6 neighbours of coefficient * e(neighbour); Dirichlet neighbours are zero
template <typename V, typename P>
__device__ __forceinline__ typename V::value_type nb_sum(const V &L, P e, int i, int j, int k) {
    using T = typename V::value_type;
    T s = 0;
    const T cx = L.cxy[k];
    if (L.nx > 1) s += cx * (e[cidx(L, wrap_p(i, L.nx), j, k)] + e[cidx(L, wrap_m(i, L.nx), j, k)]);
    if (L.ny > 1) s += cx * (e[cidx(L, i, wrap_p(j, L.ny), k)] + e[cidx(L, i, wrap_m(j, L.ny), k)]);
    if (k > 0) s += L.czm[k] * e[cidx(L, i, j, k - 1)];
    if (k < L.nz - 1) s += L.czp[k] * e[cidx(L, i, j, k + 1)];
    return s;
}

template <typename V>
__device__ __forceinline__ typename V::value_type diag_of(const V &L, int i, int j, int k) {
    typename V::value_type d = L.dg[k];
    if (has_sig(L, k)) d += L.sig[sidx(L, i, j, k)];
    return d;
}

// Gauss-Seidel update of one cell of (L + diag sigma) e = r.  Every smoother forms a value as
// (r + neighbour sum) times the reciprocal of the diagonal: the kernels that hold a level in LDS
// form the reciprocal once for all sweeps, and the others round alike (the product stays a
// product where its value feeds a sum in the same thread: no contraction).
template <typename T>
__device__ __forceinline__ T gs_value(T rhs, T diag) {
#pragma clang fp contract(off)
    return rhs * (T(1) / diag);
}
template <typename V>
__device__ __forceinline__ void gs_cell(const V &L, int i, int j, int k, int zero_init) {
    const int c = cidx(L, i, j, k);
    const auto d = diag_of(L, i, j, k);
    L.e[c] = gs_value(zero_init ? L.r[c] : L.r[c] + nb_sum(L, L.e, i, j, k), d);
}

// Colour of a cell on a plainly stored level (odd x or y extent).  With an
// odd periodic extent the parity colouring makes the wrap neighbours equal
// coloured, so the last column / row (for odd nx / ny) get colours 2 and 3:
// no two cells of one colour are then neighbours, and a sweep is the four
// colours in turn.  With both extents odd one corner is left: of a plane's cells
// (nx-1, 0), (0, ny-1) and (nx-1, ny-1), all of one colour, the last is a neighbour
// of the others.  A launched sweep then reads there either the new or the old value,
// so two runs may differ in the last bits; the coarse kernel orders the two with a barrier.
template <typename V>
__device__ __forceinline__ int nat_color(const V &L, int i, int j, int k) {
    const int par = (i + j + k) & 1;
    const bool edge = ((L.nx & 1) && i == L.nx - 1) || ((L.ny & 1) && j == L.ny - 1);
    return edge ? 2 + par : par;
}

// Residual of the finer level restricted to one coarse cell: volume-weighted
// mean over the children, likewise sigma.  On a red/black level the black
// children are skipped: right after a black half-sweep their residual is
// zero (each black equation has just been solved exactly).
// The child loops are unrolled (XY fixes their extent, a coarse plane has one
// or two children) so that a thread issues all its loads together.  XY is the
// lateral transfer mode: 0 none, 1 x and y halved, 2 x halved on a single row.
template <int XY, typename V, typename X>
__device__ __forceinline__ void restrict_cell_t(const V &F, const V &C, const X &Xf, int I, int J, int K) {
    using T = typename V::value_type;
    constexpr int nsx = XY ? 2 : 1, nsy = XY == 1 ? 2 : 1;
    double sr = 0.0, ss = 0.0;
    const int ks = Xf.cks[K], cnt = Xf.ccnt[K];
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
        if (dz >= cnt) break;
        const int k = ks + dz;
        const double wz = (double)Xf.fthick[k] / (double)Xf.cthick[K];
        const bool hs = has_sig(F, k);
#pragma unroll
        for (int dy = 0; dy < nsy; ++dy) {
            const int j = XY == 1 ? 2 * J + dy : J;
#pragma unroll
            for (int dx = 0; dx < nsx; ++dx) {
                const int i = XY ? 2 * I + dx : I;
                const T sg = hs ? F.sig[sidx(F, i, j, k)] : T(0);
                ss += wz * (double)sg;
                if (F.rb && ((i + j + k) & 1)) continue;
                const int c = cidx(F, i, j, k);
                const T res = F.r[c] - ((F.dg[k] + sg) * F.e[c] - nb_sum(F, F.e, i, j, k));
                sr += wz * (double)res;
            }
        }
    }
    const double wxy = XY == 1 ? 0.25 : (XY == 2 ? 0.5 : 1.0);
    C.r[cidx(C, I, J, K)] = (T)(sr * wxy);
    if (has_sig(C, K)) C.sig[sidx(C, I, J, K)] = (T)(ss * wxy);
}
template <typename V, typename X>
__device__ __forceinline__ void restrict_cell(const V &F, const V &C, const X &Xf, int I, int J, int K) {
    if (Xf.xy == 1) restrict_cell_t<1>(F, C, Xf, I, J, K);
    else if (Xf.xy == 2) restrict_cell_t<2>(F, C, Xf, I, J, K);
    else restrict_cell_t<0>(F, C, Xf, I, J, K);
}

// Fused multiply-add of the working precision, written out so that every kernel that
// interpolates rounds alike whatever the compiler would contract.
__device__ __forceinline__ double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Neighbour sum of a red/black cell from the other colour's six values; cx, cy (0 for a single
// row), cm and cp (0 at the contacts) weigh the x, y, lower and upper neighbours.  With the red
// residual below one expression shared by every kernel, so that they round alike.
template <typename T>
__device__ __forceinline__ T nb6(T cx, T cy, T cm, T cp, T ex0, T ex1, T ey0, T ey1, T ez0, T ez1) {
    return fmad(cp, ez1, fmad(cm, ez0, fmad(cy, ey0 + ey1, cx * (ex0 + ex1))));
}
template <typename T, int AS>
__device__ __forceinline__ T rb_nb_sum(const Lv<T, AS> &L, int k, T ex0, T ex1, T ey0, T ey1, T ez0, T ez1) {
    const T cx = L.cxy[k];
    return nb6(cx, L.ny > 1 ? cx : T(0), k > 0 ? L.czm[k] : T(0), k < L.nz - 1 ? L.czp[k] : T(0), ex0, ex1, ey0, ey1, ez0,
               ez1);
}
template <typename T>
__device__ __forceinline__ T res_value(T r, T diag, T e, T nb) { return r - fmad(diag, e, -nb); }

// The same restriction for a red/black level halved in x and y, in global
// memory, with every load issued before any arithmetic: in each child row the
// red child is the one with dx = (dy + k) & 1, a coarse plane with a single
// child reads that plane twice (the copy is skipped below), and sigma outside
// the semiconductor planes is read from the cell's own residual and ignored.
// Without conditional loads the compiler keeps all of them (48) in flight at
// once instead of waiting on each child's stencil in turn.
template <typename V, typename X>
__device__ __forceinline__ void restrict_cell_rbxy(const V &F, const V &C, const X &Xf, int I, int J, int K) {
    using T = typename V::value_type;
    const int ks = Xf.cks[K], cnt = Xf.ccnt[K];
    T sg[2][2][2], rv[2][2], ev[2][2], nb[2][2][6], cx[2], czm[2], czp[2], dg[2];
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
        const int k = ks + (dz < cnt ? dz : 0);
        const bool hs = has_sig(F, k);
        const int km = k > 0 ? k - 1 : k, kp = k < F.nz - 1 ? k + 1 : k;
        cx[dz] = F.cxy[k];
        czm[dz] = F.czm[k];
        czp[dz] = F.czp[k];
        dg[dz] = F.dg[k];
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            const int j = 2 * J + dy;
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                const int i = 2 * I + dx;
                const auto sp = hs ? F.sig + sidx(F, i, j, k) : F.r + cidx(F, i, j, k);
                sg[dz][dy][dx] = *sp;
            }
            const int i = 2 * I + ((dy + k) & 1);
            const int c = cidx(F, i, j, k);
            rv[dz][dy] = F.r[c];
            ev[dz][dy] = F.e[c];
            nb[dz][dy][0] = F.e[cidx(F, wrap_p(i, F.nx), j, k)];
            nb[dz][dy][1] = F.e[cidx(F, wrap_m(i, F.nx), j, k)];
            nb[dz][dy][2] = F.e[cidx(F, i, wrap_p(j, F.ny), k)];
            nb[dz][dy][3] = F.e[cidx(F, i, wrap_m(j, F.ny), k)];
            nb[dz][dy][4] = F.e[cidx(F, i, j, km)];
            nb[dz][dy][5] = F.e[cidx(F, i, j, kp)];
        }
    }
    double sr = 0.0, ss = 0.0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
        if (dz >= cnt) break;
        const int k = ks + dz;
        const double wz = (double)Xf.fthick[k] / (double)Xf.cthick[K];
        const bool hs = has_sig(F, k);
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                const T sgc = hs ? sg[dz][dy][dx] : T(0);
                ss = fmad(wz, (double)sgc, ss);
                if (dx != ((dy + k) & 1)) continue;
                const T nbs = nb6(cx[dz], cx[dz], k > 0 ? czm[dz] : T(0), k < F.nz - 1 ? czp[dz] : T(0), nb[dz][dy][0],
                                  nb[dz][dy][1], nb[dz][dy][2], nb[dz][dy][3], nb[dz][dy][4], nb[dz][dy][5]);
                sr = fmad(wz, (double)res_value(rv[dz][dy], dg[dz] + sgc, ev[dz][dy], nbs), sr);
            }
        }
    }
    C.r[cidx(C, I, J, K)] = (T)(sr * 0.25);
    if (has_sig(C, K)) C.sig[sidx(C, I, J, K)] = (T)(ss * 0.25);
}

// The lateral interpolant of one coarse plane: sum of w[yy][xx] v[yy][xx] in row order,
// the first term a product and the others fused multiply-adds.  With lint_z, the value
// of a fine plane from its parent plane s0 and the neighbour plane s1.  Every
// prolongation (per fine cell, fused into the red half-sweep, by coarse columns, and
// inside the coarse kernel) goes through these two, so their corrections agree bit for
// bit.
template <int NY, int NX, typename T>
__device__ __forceinline__ T lint_xy(const T (&w)[2][2], const T (&v)[2][2]) {
    T s = w[0][0] * v[0][0];
#pragma unroll
    for (int yy = 0; yy < NY; ++yy)
#pragma unroll
        for (int xx = 0; xx < NX; ++xx)
            if (yy + xx > 0) s = fmad(w[yy][xx], v[yy][xx], s);
    return s;
}
template <typename T>
__device__ __forceinline__ T lint_z(T wa, T s0, T wb, T s1) {
    return fmad(wb, s1, wa * s0);
}

// e_f += I e_c: bilinear in x,y (cell-centred 3/4, 1/4), in z linear in the
// series resistance between coarse plane centres (zero on contact faces).  On
// a red/black level only black cells are corrected: the red values are
// overwritten by the next red half-sweep without being read.
// Unrolled like the restriction: all coarse values are loaded together; a
// missing second plane (contact side) reads the first with weight zero.
// prolong_value returns the interpolated correction of fine cell (i, j, k);
// XY is the lateral transfer mode as in the restriction (2: linear in x only).
template <int XY, typename V, typename X>
__device__ __forceinline__ typename V::value_type prolong_value(const V &C, const X &Xf, int i, int j, int k) {
    using T = typename V::value_type;
    constexpr int nsx = XY ? 2 : 1, nsy = XY == 1 ? 2 : 1;
    int ix[2], jy[2];
    T wx[2], wy[2];
    if (XY == 1) {
        const int I = i >> 1, J = j >> 1;
        ix[0] = I; ix[1] = (i & 1) ? wrap_p(I, C.nx) : wrap_m(I, C.nx);
        jy[0] = J; jy[1] = (j & 1) ? wrap_p(J, C.ny) : wrap_m(J, C.ny);
        wx[0] = wy[0] = T(0.75);
        wx[1] = wy[1] = T(0.25);
    } else if (XY == 2) {
        const int I = i >> 1;
        ix[0] = I; ix[1] = (i & 1) ? wrap_p(I, C.nx) : wrap_m(I, C.nx);
        jy[0] = jy[1] = j;
        wx[0] = T(0.75);
        wx[1] = T(0.25);
        wy[0] = T(1);
        wy[1] = T(0);
    } else {
        ix[0] = ix[1] = i; jy[0] = jy[1] = j; wx[0] = wy[0] = T(1);
        wx[1] = wy[1] = T(0);
    }
    const int ka = Xf.pka[k], kb = Xf.pkb[k];
    const int kz[2] = {ka, kb >= 0 ? kb : ka};
    T w[2][2], s[2];
#pragma unroll
    for (int yy = 0; yy < 2; ++yy)
#pragma unroll
        for (int xx = 0; xx < 2; ++xx) w[yy][xx] = wx[xx] * wy[yy];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        T v[2][2] = {{T(0), T(0)}, {T(0), T(0)}};
#pragma unroll
        for (int yy = 0; yy < nsy; ++yy)
#pragma unroll
            for (int xx = 0; xx < nsx; ++xx) v[yy][xx] = C.e[cidx(C, ix[xx], jy[yy], kz[q])];
        s[q] = lint_xy<nsy, nsx>(w, v);
    }
    return lint_z(T(Xf.pwa[k]), s[0], kb >= 0 ? T(Xf.pwb[k]) : T(0), s[1]);
}
template <typename V, typename X>
__device__ __forceinline__ void prolong_cell(const V &F, const V &C, const X &Xf, int i, int j, int k) {
    if (F.rb && !((i + j + k) & 1)) return;
    F.e[cidx(F, i, j, k)] += Xf.xy == 1   ? prolong_value<1>(C, Xf, i, j, k)
                             : Xf.xy == 2 ? prolong_value<2>(C, Xf, i, j, k)
                                          : prolong_value<0>(C, Xf, i, j, k);
}

// Sum over a 256-thread block; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *lds) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int tid = threadIdx.y * blockDim.x + threadIdx.x;
    if ((tid & 63) == 0) lds[tid >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (tid == 0)
        for (int q = 0; q < (int)((blockDim.x * blockDim.y) >> 6); ++q) s += lds[q];
    return s;
}

// phi buffer holding the input / output of the cycle in progress (cycle c = cycles)
__device__ __forceinline__ int cyc_src(const GState *s) {
    return s->cycles == 0 ? s->start : ((s->cycles - 1) % 2 == 0 ? s->oth0 : s->oth1);
}
__device__ __forceinline__ int cyc_dst(const GState *s) { return s->cycles % 2 == 0 ? s->oth0 : s->oth1; }

// ------------------------------------------------------------------- TDGL
// eq. (TDGL2) with forward Euler (Step 1a); surface stencils of eqs. (Pbc),
// (PbcFree), (PbcDir) on the two ferroelectric boundary planes.
__device__ __forceinline__ double surface_value(int pbc, double lambda, double h, double p0, double p1) {
    if (pbc == 0) return (9.0 * p0 - p1) * 0.125;
    if (pbc == 1) return 0.0;
    return lambda * (9.0 * p0 - p1) / (8.0 * lambda + 3.0 * h);
}

// The variational force dF/dP of eq. (TDGL2) at cell (i, j, k), c its index;
// the time derivative is -Gamma times it.
template <typename T>
__device__ __forceinline__ double tdgl_force(const Inst<T> &a, const double FX_AS(1) *P,
                                             const double FX_AS(1) *phi, int i, int j, int k, size_t c) {
    const size_t nxy = (size_t)a.nx * a.ny;
    const double h = a.h, ih2 = 1.0 / (h * h), i2h = 0.5 / h;
    const double p = P[c];
    const size_t row = c - i;
    const double dxx = (P[row + wrap_p(i, a.nx)] - 2.0 * p + P[row + wrap_m(i, a.nx)]) * ih2;
    const size_t pl = (size_t)k * nxy + i;
    const double dyy = (P[pl + (size_t)wrap_p(j, a.ny) * a.nx] - 2.0 * p + P[pl + (size_t)wrap_m(j, a.ny) * a.nx]) * ih2;
    double dzz, dphi;
    if (k == a.f0) {
        const double p1 = P[c + nxy];
        dzz = 4.0 * (2.0 * surface_value(a.pbc, a.lambda, h, p, p1) - 3.0 * p + p1) * ih2 * (1.0 / 3.0);
        dphi = (-3.0 * phi[c] + 4.0 * phi[c + nxy] - phi[c + 2 * nxy]) * i2h;
    } else if (k == a.f1 - 1) {
        const double p1 = P[c - nxy];
        dzz = 4.0 * (2.0 * surface_value(a.pbc, a.lambda, h, p, p1) - 3.0 * p + p1) * ih2 * (1.0 / 3.0);
        dphi = (3.0 * phi[c] - 4.0 * phi[c - nxy] + phi[c - 2 * nxy]) * i2h;
    } else {
        dzz = (P[c + nxy] - 2.0 * p + P[c - nxy]) * ih2;
        dphi = (phi[c + nxy] - phi[c - nxy]) * i2h;
    }
    const double p2 = p * p;
    const double landau = p * (a.alpha + p2 * (a.beta + a.gamma * p2));
    return landau - a.g44 * (dxx + dyy) - a.g11 * dzz + dphi;
}

// The update of one tile: P^{n+1} into dst.  Euler (Step 1a): src + dt f(src, phi^n).
// Corrector (Step 2a): P^{n+1} = P^n + dt/2 f(P^n, phi^n) + dt/2 f(P*, phi*); with
// P* = P^n + dt f(P^n, phi^n) this is (P^n + P*)/2 + dt/2 f(P*, phi*).  There src holds P*
// and dst P^n, overwritten in place (each cell reads only its own).
template <typename T>
__device__ __forceinline__ void tdgl_tile(const Inst<T> &a, const GState *s, int tile, int src, int corr) {
    const T3 t = split3(tile, a.nx, a.ny);
    const int i = t.tx * BX + threadIdx.x;
    const int j = t.ty * BY + threadIdx.y;
    const int k = a.f0 + t.tz;
    if (i >= a.nx || j >= a.ny) return;
    const size_t c = ((size_t)k * a.ny + j) * a.nx + i;
    const double FX_AS(1) *P = asp<1>(a.P[src]);
    double FX_AS(1) *out = asp<1>(a.P[1 - src]);
    const double dF = tdgl_force(a, P, asp<1>(a.phi[s->cur]), i, j, k, c);
    if (corr) out[c] = 0.5 * (out[c] + P[c]) - 0.5 * s->dt * a.Gamma * dF;
    else out[c] = P[c] - s->dt * a.Gamma * dF;
}

// A stand-alone Euler update of every instance (the P buffers are flipped after it).
template <typename T>
__global__ __launch_bounds__(256) void k_tdgl(const Inst<T> *I, Work w) {
    const Blk b = find_block(w);
    if (!b.ok) return;
    const GState *s = wstate(w, b.inst);
    tdgl_tile(I[b.inst], s, b.t, s->pcur, 0);
}

// ------------------------------------------------------- solve bookkeeping
// After a stand-alone TDGL update: the new P is in the other buffer, and the
// stored time levels no longer belong to one time series.
template <typename T>
__global__ void k_flip(const Inst<T> *I, int ninst) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= ninst) return;
    GState *s = asp<1>(I[n].st);
    s->pcur ^= 1;
    s->hist = 0;
}

// Start a solve of one instance, its state in registers.  sel = 1 (time step, instances
// flagged by the advance slot): the P update this slot computes becomes the current P, the
// gate potential vg comes from the run's schedule (has_v), and the starting iterate may be
// extrapolated in time.  sel = 0: a plain solve from its current phi.
template <typename T>
__device__ __forceinline__ void begin_solve(const Inst<T> &a, InstState *s, int sel, bool has_v, double vg) {
    if (sel) {
        s->pcur ^= 1;
        if (s->adv && has_v) s->v_top = vg;
    } else {
        s->phase = 0;
        s->pstar = -1;
    }
    // A corrector's solve starts from the predictor's phi*, O(dt^2) away from phi^{n+1},
    // unless the history through phi^n supports an extrapolation of order >= 2, which is
    // O(dt^3) away or closer.  A predictor's target phi* differs from phi^{n+1} by a
    // smooth O(dt^2) offset: with the last step's phi* kept, it starts from the
    // extrapolation plus that step's offset phi*_n - phi^n, O(dt^3) away.
    int order = 0;
    if (sel && s->adv) order = min(s->hist, a.warm);
    else if (sel) order = min(s->hist - 1, a.warm) >= 2 ? min(s->hist - 1, a.warm) : 0;
    const int usestar = sel && s->adv && a.order2 && s->pstar >= 0;
    if (!usestar) s->pstar = -1;
    int o0 = 0, o1 = 0, no = 0;
#pragma unroll
    for (int q = 0; q < kPhiBufs; ++q) {
        bool used = q >= a.nbuf || q == s->cur || q == s->pstar;
#pragma unroll
        for (int m = 0; m < kMaxHist; ++m) used |= m < s->hist && s->prev[m] == q;
        if (!used) {
            if (no == 0) o0 = q;
            else if (no == 1) o1 = q;
            ++no;
        }
    }
    s->oth0 = o0;
    s->oth1 = o1;
    s->order = order;
    s->usestar = usestar;
    const int cur = s->cur;
    s->start = order > 0 || usestar ? o1 : cur;
    s->ts = sel;
    s->done = 0;
    s->cycles = 0;
    s->zpend = 0;
    s->fresh = 1;
    s->insolve = 1;
    s->light = 0;
}

// One thread per instance: start the solves (after k_head in the first advance slot of a
// run, or a plain solve of every instance).
template <typename T>
__global__ void k_begin(const Inst<T> *I, InstState *S, int ninst, int sel) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= ninst) return;
    const Inst<T> &a = I[n];
    GState *gs = asp<1>(S + n);
    InstState st = *(const InstState *)gs, *s = &st;
    if (sel && !s->adv && !s->corr) return;
    const int q = s->step - s->sched_base;
    const bool has_v = sel && s->adv && q >= 0 && q < s->sched_len;
    begin_solve(a, s, sel, has_v, has_v ? asp<1>(a.vsched)[q] : 0.0);
    *(InstState *)gs = st;
}

// Lagrange extrapolation to t^{n+1} through t^n, t^{n-1}, ... (equal steps).
__device__ constexpr double kExtrapC[4][4] = {{1, 0, 0, 0}, {2, -1, 0, 0}, {3, -3, 1, 0}, {4, -6, 4, -1}};

// Four cells per thread, every load ahead of the first store (the levels could alias the
// output as far as the compiler knows, so a cell's store would hold up the next cell's loads).
template <int ORD, int STAR>
__device__ __forceinline__ void extrap_cells(const double FX_AS(1) *const (&in)[4], const double FX_AS(1) *star,
                                             double FX_AS(1) *out, size_t base, size_t n) {
    constexpr int U = kExtrapChunk / 256;
    const size_t c0 = base + threadIdx.y * BX + threadIdx.x;
    double x[ORD + 1][U], sv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t c = min(c0 + 256 * u, n - 1);
#pragma unroll
        for (int m = 0; m <= ORD; ++m) x[m][u] = in[m][c];
        if (STAR) sv[u] = star[c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        double v = kExtrapC[ORD][0] * x[0][u];
#pragma unroll
        for (int m = 1; m <= ORD; ++m) v = fmad(kExtrapC[ORD][m], x[m][u], v);
        if (STAR) v += sv[u] - x[0][u];
        if (c0 + 256 * u < n) out[c0 + 256 * u] = v;
    }
}

template <typename T>
__device__ __forceinline__ void extrap_tile(const Inst<T> &a, const GState *s, int tile) {
    const int order = s->order, usestar = s->usestar;
    const size_t nxy = (size_t)a.nx * a.ny, off = (size_t)a.kb * nxy, n = (size_t)a.nzd * nxy;
    // newest level phi^n: the current iterate, or for a corrector the last stored level
    const int sh = s->phase == 1 ? 1 : 0;
    const int cur = s->cur, pstar = s->pstar, start = s->start;
    const int p0 = s->prev[0], p1 = s->prev[1], p2 = s->prev[2], p3 = s->prev[3];
    const double FX_AS(1) *in[4] = {asp<1>(a.phi[sh ? p0 : cur]) + off, asp<1>(a.phi[sh ? p1 : p0]) + off,
                                    asp<1>(a.phi[sh ? p2 : p1]) + off, asp<1>(a.phi[sh ? p3 : p2]) + off};
    const double FX_AS(1) *star = asp<1>(a.phi[usestar ? pstar : cur]) + off;
    double FX_AS(1) *out = asp<1>(a.phi[start]) + off;
    const size_t base = (size_t)tile * kExtrapChunk;
    if (usestar) {
        if (order == 3) extrap_cells<3, 1>(in, star, out, base, n);
        else if (order == 2) extrap_cells<2, 1>(in, star, out, base, n);
        else if (order == 1) extrap_cells<1, 1>(in, star, out, base, n);
        else extrap_cells<0, 1>(in, star, out, base, n);
    } else {
        if (order == 3) extrap_cells<3, 0>(in, star, out, base, n);
        else if (order == 2) extrap_cells<2, 0>(in, star, out, base, n);
        else extrap_cells<1, 0>(in, star, out, base, n);
    }
}

// Finalize the solve of one instance (its state in registers) if it has stopped: its last
// iterate becomes phi^{n+1} and, after a successful time step, phi^n the newest stored level;
// the statistics and the status are recorded.  With advance set (an advance slot of a run),
// an instance that is idle and below its run target (and whose last solve succeeded) is
// flagged to start the next time step in this slot; one that has reached the target or
// failed is parked.
__device__ __forceinline__ void finish_solve(InstState *s, int order2, int advance) {
    int zf = 0, corr = 0, stepped = 0;
    if (s->insolve && s->done != 0) {
        const int c = s->cycles;
        s->solves += 1;
        s->total_cycles += c;
        s->max_cycles_step = max(s->max_cycles_step, c);
        s->insolve = 0;
        s->v_done = s->v_top;
        if (s->done == 2) {                   // non-finite: keep phi^n, drop the history
            s->status = 5;
            s->failed += 1;
            s->hist = 0;
        } else {
            // plain values in the conditional: one of members yields a member's address, and
            // an address taken keeps the whole state in scratch memory
            const int i0 = s->start, o0 = s->oth0, o1 = s->oth1;
            const int fin = c == 0 ? i0 : ((c - 1) % 2 == 0 ? o0 : o1);
            s->status = s->done == 1 ? 0 : 4;
            if (s->status != 0) s->failed += 1;
            const bool ok_step = s->ts && s->status == 0;
            if (ok_step && s->phase == 1) {
                // corrector done: phi^{n+1}; the predictor's phi* is kept for the next
                // predictor's start, phi^n stays the newest stored level
                s->step += 1;
                s->phase = 0;
                stepped = 1;
                s->pstar = s->cur;
            } else if (ok_step) {
                // Euler step, or the predictor of a second-order step: phi^n
                // becomes the newest stored level
                if (fin != s->cur) {
                    // Euler keeps 3 levels; a predictor-corrector instance 4, so that
                    // its corrector, whose newest level is phi^n, extrapolates cubically
                    const int hmax = order2 ? kMaxHist : kMaxHist - 1;
#pragma unroll
                    for (int m = kMaxHist - 1; m > 0; --m)
                        if (m < hmax) s->prev[m] = s->prev[m - 1];
                    s->prev[0] = s->cur;
                    s->hist = min(s->hist + 1, hmax);
                } else {
                    s->hist = 0;
                }
                if (order2) { s->phase = 1; corr = 1; }
                else { s->step += 1; stepped = 1; }
                s->pstar = -1;
            } else {
                s->hist = 0;
                s->phase = 0;
                s->pstar = -1;
            }
            s->cur = fin;
            zf = s->done == 1 && s->zpend;
        }
    }
    s->zero_fix = zf;
    int adv = 0;
    if (advance && !s->parked && !s->insolve && !corr) {
        if (s->status != 0 || s->step >= s->target) s->parked = 1;
        else adv = 1;
    }
    s->adv = adv;
    s->corr = corr;
    s->stepped = stepped;
}

// The same as a launch of its own, one thread per instance (a plain solve's end, a run's
// first advance slot).
template <typename T>
__global__ void k_head(const Inst<T> *I, InstState *S, int ninst, int advance) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= ninst) return;
    // the state is read whole, updated in registers and written back once (one
    // round trip instead of one per dependent field); the copies go through a generic
    // view (the implicit copy operations take no address-space-qualified operand),
    // which the compiler maps back to global loads and stores
    GState *gs = asp<1>(S + n);
    InstState st = *(const InstState *)gs;
    finish_solve(&st, I[n].order2, advance);
    *(InstState *)gs = st;
}

// Q-V diagnostics (Results, MFIM).  Across the ferroelectric/dielectric face, with L
// the lower and R the upper plane, the Poisson operator's flux is
// D = -eps_f (phi_R - phi_L)/h + P_f (harmonic-mean eps_f, P_f = (eps_R P_L + eps_L P_R)
// / (eps_L + eps_R)), equal to eps0 eps_DE E_z in the dielectric half cell.  The face
// potential follows from the lower half cell, D = -eps_L (phi_int - phi_L)/(h/2) + P_L.
// Each block sums D and phi_int over a strided share of the face (fixed order), then
// a tree in LDS; the finishing kernel adds the blocks' sums in block order.
template <typename T>
__device__ __forceinline__ void qv_part_block(const Inst<T> &a, const GState *s, int blk, int pbuf, double (*red)[256]) {
    const int tid = threadIdx.y * blockDim.x + threadIdx.x;
    const size_t nxy = (size_t)a.nx * a.ny;
    const double FX_AS(1) *phL = asp<1>(a.phi[s->cur]) + (size_t)a.qv_kl * nxy;
    const double FX_AS(1) *phR = phL + nxy;
    const double FX_AS(1) *Pfe = asp<1>(a.P[pbuf]) + (size_t)(a.qv_kl + a.qv_fe_up) * nxy;
    const double eL = a.qv_el, eR = a.qv_er, ih = 1.0 / a.h;
    const double ef = 2.0 * eL * eR / (eL + eR), wL = eR / (eL + eR), wR = eL / (eL + eR);
    const double hh_eL = 0.5 * a.h / eL;
    double sd = 0.0, sp = 0.0;
    for (size_t c = (size_t)blk * 256 + tid; c < nxy; c += (size_t)kQvBlocks * 256) {
        const double p = Pfe[c];
        const double pL = a.qv_fe_up ? 0.0 : p, pR = a.qv_fe_up ? p : 0.0;
        const double D = -ef * (phR[c] - phL[c]) * ih + wL * pL + wR * pR;
        sd += D;
        sp += phL[c] - (D - pL) * hh_eL;
    }
    red[0][tid] = sd;
    red[1][tid] = sp;
    __syncthreads();
    for (int m = 128; m > 0; m >>= 1) {
        if (tid < m) {
            red[0][tid] += red[0][tid + m];
            red[1][tid] += red[1][tid + m];
        }
        __syncthreads();
    }
    if (tid == 0) {
        double FX_AS(1) *o = asp<1>(a.qv_part) + 2 * blk;
        o[0] = red[0][0];
        o[1] = red[1][0];
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_qv_part(const Inst<T> *I) {
    __shared__ double red[2][256];
    const Inst<T> &a = I[blockIdx.x / kQvBlocks];
    const GState *s = asp<1>(a.st);
    if (a.qv_kl < 0) return;
    qv_part_block(a, s, blockIdx.x % kQvBlocks, s->pcur, red);
}

// Q and V_fe from the face sums, with gate potential vt.
template <typename T>
__device__ __forceinline__ void qv_finish(const Inst<T> &a, double vt, double &Q, double &V) {
    double sd = 0.0, sp = 0.0;
    const double FX_AS(1) *p = asp<1>(a.qv_part);
    for (int b = 0; b < kQvBlocks; ++b) { sd += p[2 * b]; sp += p[2 * b + 1]; }
    const double area = (double)a.nx * a.ny;
    Q = -sd / area;
    V = vt - sp / area;
}

template <typename T>
__global__ void k_qv_fin(const Inst<T> *I, int ninst, double *out) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= ninst) return;
    const Inst<T> &a = I[n];
    double Q = __builtin_nan(""), V = __builtin_nan("");
    if (a.qv_kl >= 0) qv_finish(a, asp<1>(a.st)->v_top, Q, V);
    asp<1>(out)[2 * n] = Q;
    asp<1>(out)[2 * n + 1] = V;
}

// The field work of an advance slot, after the states have moved on: the TDGL update (Euler or
// corrector) of the instances whose P buffers were flipped, the starting iterate of the
// solves just begun, and, when a run records Q and V_fe, the face sums of the steps just
// completed (their P is the buffer the flip left behind).  The three parts read and write
// different buffers, so they can share a launch.  Grid: gt blocks of TDGL tiles, ge of
// extrapolation tiles, the rest face sums; PART names the parts a launch holds (1 TDGL, 2 the
// others, 3 all): see launch_fields.
template <typename T, int PART>
__global__ __launch_bounds__(256) void k_fields(const Inst<T> *I, Work wt, Work we, int gt, int ge) {
    __shared__ double red[2][256];
    const int bx = blockIdx.x;
    if ((PART & 1) && bx < gt) {
        const Blk b = find_block(wt, bx, gt);
        const GState *s = wstate(wt, b.inst);
        const int adv = s->adv, corr = s->corr;
        if (!b.ok | ((adv == 0) & (corr == 0))) return;  // one exit test: see smooth_kernel
        tdgl_tile(I[b.inst], s, b.t, 1 - s->pcur, corr);
    } else if ((PART & 2) && bx < gt + ge) {
        const Blk b = find_block(we, bx - gt, ge);
        const GState *s = wstate(we, b.inst);
        const int order = s->order, fresh = s->fresh, usestar = s->usestar;
        if (!b.ok | (fresh == 0) | ((order == 0) & (usestar == 0))) return;
        extrap_tile(I[b.inst], s, b.t);
    } else if (PART & 2) {
        const int q = bx - gt - ge, inst = q / kQvBlocks;
        const Inst<T> &a = I[inst];
        const GState *s = asp<1>(wt.st + inst);
        if ((a.qv_kl < 0) | (s->stepped == 0)) return;
        qv_part_block(a, s, q % kQvBlocks, s->adv ? 1 - s->pcur : s->pcur, red);
    }
}

// ------------------------------------------------------ fine-level residual
// Per-plane tables of the finest level the residual reads (scaled by h^2/eps0).
struct ResTab {
    const double FX_AS(1) *cxy, *czm, *czp, *wl, *wr, *p0e, *n0e;
};
template <typename T>
__device__ __forceinline__ ResTab res_tab(const Inst<T> &a) {
    return ResTab{asp<1>(a.cxy0), asp<1>(a.czm0), asp<1>(a.czp0), asp<1>(a.wl), asp<1>(a.wr), asp<1>(a.p0e),
                  asp<1>(a.n0e)};
}

// One device cell of plane k (eq. (Poisson) with eq. (rho), scaled by h^2/eps0): the
// right-hand side f (contact terms and the bound charge -(P_f(k+1/2) - P_f(k-1/2))/h),
// the residual r = f - N(phi) and the Newton sigma = -d rho_c/d phi (semiconductor
// planes).  v0 is the cell's phi, vx0/vx1 and vy0/vy1 its x+1/x-1 and y+1/y-1
// neighbours, vzm/vzp its z neighbours (not used on the contact planes), pm/pc/pp P on
// planes k-1, k, k+1 (read only where a polarised face touches the plane).  Fused
// multiply-adds are written out, so that every residual kernel rounds alike.  FD = 0
// leaves the Fermi-Dirac branch out (launches whose instances all take Boltzmann carriers:
// fewer registers, no scalar registers parked in vector lanes).
template <typename T, int FD>
__device__ __forceinline__ void res_cell(const Inst<T> &a, const ResTab &tb, int k, int nzd, int fl, double v_t,
                                        double v0, double vx0, double vx1, double vy0, double vy1, double vzm,
                                        double vzp, double pm, double pc, double pp, double &f_o, double &r_o,
                                        double &sg_o) {
    const double nb = fmad(-2.0, v0, vx0 + vx1) + fmad(-2.0, v0, vy0 + vy1);
    const double dn = k > 0 ? vzm : 0.0;
    const double up = k < nzd - 1 ? vzp : 0.0;
    const double Lphi = fmad(tb.czp[k], v0 - up, fmad(tb.czm[k], v0 - dn, -tb.cxy[k] * nb));
    double f = 0.0;
    if (fl & PF_P) {
        const double pup = k == nzd - 1 ? pc : fmad(tb.wr[k], pp, tb.wl[k] * pc);
        const double pdn = k == 0 ? pc : fmad(tb.wr[k - 1], pc, tb.wl[k - 1] * pm);
        f = -(pup - pdn) * a.p_scale;
    }
    if (k == 0) f = fmad(tb.czm[k], a.v_b, f);
    if (k == nzd - 1) f = fmad(tb.czp[k], v_t, f);
    double r = f - Lphi, sg = 0.0;
    if (fl & PF_SC) {
        const double u = v0 * a.vt_inv;
        const double p0e = tb.p0e[k], n0e = tb.n0e[k];
        if (FD && a.fd) {
            // differences from the neutral state: rho_c(0) = 0 exactly
            const double FX_AS(1) *ft = asp<1>(a.fdt) + 4 * k;
            double Fp, dFp, Fn, dFn;
            fd_half(ft[0] - u, Fp, dFp);
            fd_half(ft[1] + u, Fn, dFn);
            r = fmad(fmad(p0e, Fp - ft[2], -(n0e * (Fn - ft[3]))), a.rho_scale, r);
            sg = fmad(p0e, dFp, n0e * dFn) * a.sig_scale;
        } else {
            // e^u - 1 and e^-u - 1 from one expm1: with t = e^|u| - 1 the other
            // is -t / (1 + t), free of cancellation for either sign of u
            const double t1 = expm1(fabs(u));
            const double t2 = -t1 / (1.0 + t1);
            const double ep = u >= 0.0 ? t1 : t2, em = u >= 0.0 ? t2 : t1;
            r = fmad(fmad(p0e, em, -(n0e * ep)), a.rho_scale, r);           // + rho_c
            sg = fmad(p0e, 1.0 + em, n0e * (1.0 + ep)) * a.sig_scale;
        }
    }
    f_o = f;
    r_o = r;
    sg_o = sg;
}

// Each thread owns a column of kResZ planes.  All loads are issued before any
// arithmetic (clamped indices instead of boundary branches; the column's
// z-neighbours are loaded once) and all stores follow it, so a wave makes one
// memory round trip for kResZ cells.  Mode 0 evaluates the current iterate; mode 2 (update not
// folded into the smoother) first forms phi_out = phi_in + clip(e).
template <typename T, int MODE, int FD>
__device__ __forceinline__ void residual_body(const Inst<T> &a, const GState *s, const T3 &t, int after_cycle,
                                              double &rr, double &ff) {
    const int ZT = kResZ;
    const int nx = a.nx, ny = a.ny, nzd = a.nzd;
    const int ii = t.tx * BX + threadIdx.x;
    const int jj = t.ty * BY + threadIdx.y;
    const bool live = ii < nx && jj < ny;
    const int i = live ? ii : 0, j = live ? jj : 0;
    const int k0 = t.tz * ZT;
    const int nxy = nx * ny;
    const size_t off = (size_t)a.kb * nxy;
    const int bin = MODE == 2 ? cyc_src(s) : (after_cycle ? cyc_dst(s) : s->start);
    const double FX_AS(1) *phi = asp<1>(a.phi[bin]) + off;
    double FX_AS(1) *phi_out = asp<1>(a.phi[cyc_dst(s)]) + off;
    const double FX_AS(1) *P = asp<1>(a.P[s->pcur]) + off;
    const Lv<T, 1> L = gview(a.lv[0]);
    const int FX_AS(1) *pflags = asp<1>(a.pflags);
    const int col = j * nx + i;
    const int ox0 = wrap_p(i, nx) - i, ox1 = wrap_m(i, nx) - i;
    const int oy0 = (wrap_p(j, ny) - j) * nx, oy1 = (wrap_m(j, ny) - j) * nx;
    const int rb = L.rb;
    const int half = (nxy * nzd) >> 1;
    const double big = 1e300;
    auto kcl = [&](int k) { return k < 0 ? 0 : (k >= nzd ? nzd - 1 : k); };
    int fl[ZT];
#pragma unroll
    for (int z = 0; z < ZT; ++z) fl[z] = pflags[kcl(k0 + z)];
    bool anyP = false;
#pragma unroll
    for (int z = 0; z < ZT; ++z) anyP |= (k0 + z < nzd) && (fl[z] & PF_P);
    // P is read only by columns that hold a polarised plane; the others load
    // the phi cells they read anyway (cache hits, values unused), so that no
    // branch joins ahead of the phi loads and every load is in flight at once.
    const double FX_AS(1) *Psrc = anyP ? P : phi;
    double pz[ZT + 2];
#pragma unroll
    for (int z = 0; z < ZT + 2; ++z) pz[z] = Psrc[kcl(k0 - 1 + z) * nxy + col];
    double vc[ZT + 2], vx0[ZT], vx1[ZT], vy0[ZT], vy1[ZT];
    auto at = [&](int k, int o, int par, double *dst) {
        const int c = k * nxy + col + o;
        double v = phi[c];
        if (MODE == 2) {
            const double d = (double)L.e[rb ? (par ? half : 0) + (c >> 1) : c];
            const double lim = (pflags[k] & PF_SC) ? a.dmax : big;
            v += fmin(fmax(d, -lim), lim);
        }
        *dst = v;
    };
    const int par0 = (i + j) & 1;
#pragma unroll
    for (int z = 0; z < ZT + 2; ++z) {
        const int k = kcl(k0 - 1 + z);
        at(k, 0, par0 ^ (k & 1), &vc[z]);
    }
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = kcl(k0 + z);
        const int pn = par0 ^ (k & 1) ^ 1;
        // one row (ny = 1): the y neighbours are the cell itself, of its own colour, so
        // that their terms cancel as in the operator
        const int py = ny > 1 ? pn : pn ^ 1;
        at(k, ox0, pn, &vx0[z]);
        at(k, ox1, pn, &vx1[z]);
        at(k, oy0, py, &vy0[z]);
        at(k, oy1, py, &vy1[z]);
    }
    const double v_t = s->v_top;
    const ResTab tb = res_tab(a);
    double res[ZT], sg[ZT];
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = k0 + z;
        res[z] = 0.0;
        sg[z] = 0.0;
        if (k >= nzd) break;
        double f;
        res_cell<T, FD>(a, tb, k, nzd, fl[z], v_t, vc[z + 1], vx0[z], vx1[z], vy0[z], vy1[z], vc[z], vc[z + 2], pz[z],
                 pz[z + 1], pz[z + 2], f, res[z], sg[z]);
        if (live) {
            rr = fmad(res[z], res[z], rr);
            ff = fmad(f, f, ff);
        }
    }
    if (!live) return;
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = k0 + z;
        if (k >= nzd) break;
        if (MODE == 2) phi_out[k * nxy + col] = vc[z + 1];
        if (fl[z] & PF_SC) L.sig[sidx(L, i, j, k)] = (T)sg[z];
        L.r[cidx(L, i, j, k)] = (T)res[z];
    }
}

// MODE 0 covers every instance except, after a cycle, those whose update is
// not folded into the smoother; MODE 2 covers exactly those (two kernels
// rather than one branch: each keeps its own, smaller register budget).
template <typename T, int MODE, int FD>
__global__ __launch_bounds__(256) void k_residual(const Inst<T> *I, Work w, int after_cycle) {
    __shared__ double lds_r[4];
    __shared__ double lds_f[4];
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const GState *s = wstate(w, b.inst);
    // one exit test: see smooth_kernel
    const int done = s->done, fresh = s->fresh, fold = a.fold;
    if (!b.ok | (after_cycle ? done != 0 : fresh == 0) | ((MODE == 2) != ((after_cycle != 0) & (fold == 0)))) return;
    // tiles walk each column up in z (halo planes shared through L2); the partial sums
    // keep the x-fastest tile index, so the reduction's order does not depend on it
    const int nzt = (a.nzd + kResZ - 1) / kResZ;
    const T3 t = split3z(b.t, a.nx, nzt);
    const int tl = t.tx + ((a.nx + BX - 1) / BX) * (t.ty + ((a.ny + BY - 1) / BY) * t.tz);
    double rr = 0.0, ff = 0.0;
    residual_body<T, MODE, FD>(a, s, t, after_cycle, rr, ff);
    const double sr = block_sum(rr, lds_r);
    const double sf = block_sum(ff, lds_f);
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        double FX_AS(1) *part = asp<1>(a.part);
        part[2 * tl] = sr;
        part[2 * tl + 1] = sf;
    }
}

// Deterministic final sum of one instance's residual partials (a block per
// instance) and its stop decision.  f = 0 exactly with a nonzero residual: N(0) = 0,
// so phi = 0 is the root; the block sets the solve's last iterate to it at once
// (the slot that finalizes the solve reads that buffer as phi^{n+1}).
// MODE 0: the residual of a solve's starting iterate; with rec the block also writes the
// (Q, V_fe) record of the step completed in this slot.  MODE 1: after a cycle.  MODE 2: after
// a cycle of a run; the block then finalizes the solve if it has stopped and starts the
// instance's next one, all on the state in thread 0's registers (launches of their own for
// these single-thread steps cost a gap of the stream each).
template <typename T, int MODE>
__global__ __launch_bounds__(1024) void k_reduce(const Inst<T> *I, InstState *S, int rec) {
    __shared__ double lr[16];
    __shared__ double lf[16];
    __shared__ int lz;
    const Inst<T> &a = I[blockIdx.x];
    GState *gs = asp<1>(S + blockIdx.x);
    // the state and the partials are read together, the partials two per thread at a
    // time, so that the block waits on memory once for them (an instance that is not
    // reduced here ignores what it read); each thread still adds its partials in
    // index order
    const double FX_AS(1) *part = asp<1>(a.part);
    const bool skip = MODE ? gs->done != 0 : !gs->fresh;
    InstState st = *(const InstState *)gs, *s = &st;
    const double tol2 = a.tol2, light_r2 = a.light_r2, light_c2 = a.light_c2;
    const int max_cycles = a.max_cycles, light_ok = a.light_ok;
    // gate potentials of the step in progress and of the one after it
    const int q0 = s->step - s->sched_base, qn = s->sched_len;
    double v0 = 0.0, v1 = 0.0;
    if (MODE == 2 && threadIdx.x == 0) {
        const double FX_AS(1) *vs = asp<1>(a.vsched);
        v0 = vs[q0 >= 0 && q0 < qn ? q0 : 0];
        v1 = vs[q0 + 1 >= 0 && q0 + 1 < qn ? q0 + 1 : 0];
    }
    const int n = tiles3(a.nx, a.ny, (a.nzd + kResZ - 1) / kResZ);
    const int B = blockDim.x;
    double r = 0.0, f = 0.0;
    int q = threadIdx.x;
    for (; q + B < n; q += 2 * B) {
        const double r0 = part[2 * q], f0 = part[2 * q + 1];
        const double r1 = part[2 * (q + B)], f1 = part[2 * (q + B) + 1];
        r += r0;
        f += f0;
        r += r1;
        f += f1;
    }
    if (q < n) { r += part[2 * q]; f += part[2 * q + 1]; }
    if (MODE == 0 && rec && threadIdx.x == 0 && a.qv_kl >= 0 && s->stepped) {
        const int qr = s->step - 1 - s->sched_base;
        if (qr >= 0 && qr < kRecSteps) {
            double Q, V;
            qv_finish(a, s->v_done, Q, V);
            double FX_AS(1) *o = asp<1>(a.qv_rec) + 2 * qr;
            o[0] = Q;
            o[1] = V;
        }
    }
    if (MODE != 2 && skip) return;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { r += __shfl_down(r, off, 64); f += __shfl_down(f, off, 64); }
    if ((threadIdx.x & 63) == 0) { lr[threadIdx.x >> 6] = r; lf[threadIdx.x >> 6] = f; }
    __syncthreads();
    if (threadIdx.x == 0) {
        int zb = -1;
        if (!skip) {
            double x = 0.0, y = 0.0;
            for (int u = 0; u < (int)(blockDim.x >> 6); ++u) { x += lr[u]; y += lf[u]; }
            const double x_prev = s->rn2;
            const int cycles = s->cycles + (MODE ? 1 : 0);
            // the solve's last iterate: the start before any cycle, else the latest cycle's output
            const int i0 = s->start, out0 = s->oth0, out1 = s->oth1;
            const int fin = cycles == 0 ? i0 : ((cycles - 1) % 2 == 0 ? out0 : out1);
            s->rn2 = x;
            s->fn2 = y;
            s->fresh = 0;
            s->cycles = cycles;
            if (!isfinite(x) || !isfinite(y)) s->done = 2;
            else if (y == 0.0) {
                s->done = 1;
                s->zpend = x != 0.0;
                if (x != 0.0) zb = fin;
            }
            else if (x <= tol2 * y || x == 0.0) s->done = 1;
            else if (cycles >= max_cycles) s->done = 3;
            // within kLightRatio of the tolerance, after a cycle that contracted the
            // residual at least kLightContraction-fold (the linear regime, as in a
            // time step's first cycle), one V(1,1)-like cycle (contraction about 0.2)
            // finishes the solve at a little over half the cost
            s->light = light_ok && MODE && x <= light_r2 * tol2 * y && x * light_c2 <= x_prev;
        }
        if (MODE == 2) {
            finish_solve(s, a.order2, 1);
            if (s->adv || s->corr) {
                const int qs = s->step - s->sched_base;
                begin_solve(a, s, 1, qs >= 0 && qs < qn, qs == q0 ? v0 : v1);
            }
            *(InstState *)gs = st;
        } else {
            gs->rn2 = s->rn2;
            gs->fn2 = s->fn2;
            gs->fresh = 0;
            gs->cycles = s->cycles;
            gs->done = s->done;
            gs->zpend = s->zpend;
            gs->light = s->light;
        }
        lz = zb;
    }
    __syncthreads();
    const int zb = lz;
    if (zb >= 0) {
        const size_t nxy = (size_t)a.nx * a.ny, nn = (size_t)a.nzd * nxy;
        double FX_AS(1) *out = asp<1>(a.phi[zb]) + (size_t)a.kb * nxy;
        for (size_t c = threadIdx.x; c < nn; c += blockDim.x) out[c] = 0.0;
    }
}

// ----------------------------------------------------------------- smoother
// One colour of red-black Gauss-Seidel on (L + diag sigma) e = r.  Split
// storage: a thread per cell of that colour, ZT planes per thread with all
// loads issued first; plainly stored levels: a thread per cell and ZT planes
// of a tile.  UPD (finest level, last black half-sweep, instances whose
// update is folded in) also writes phi_out = phi_in + clip(e) for each black
// cell and its red partner (the pair 2m, 2m+1 of a row).
template <typename T, int ZI, int ZT, int UPD>
__device__ __forceinline__ void smooth_rb_body(const Inst<T> &a, const GState *st, const Lv<T, 1> &L, int t, int color, int lbx) {
    const int hx = L.nx >> 1;
    const T3 tt = split3r(t, hx, L.ny, lbx);
    const int mm = (tt.tx << lbx) + (threadIdx.x & ((1 << lbx) - 1));
    const int jj = (tt.ty << (8 - lbx)) + (threadIdx.x >> lbx);
    const bool live = mm < hx && jj < L.ny;
    const int m = live ? mm : 0, j = live ? jj : 0;           // (0, 0): see the stores
    const int half = (L.nx * L.ny * L.nz) >> 1;
    const int plane = L.ny * hx;
    const T FX_AS(1) *eo = L.e + (color ? 0 : half);
    T FX_AS(1) *es = L.e + (color ? half : 0);
    const T FX_AS(1) *rs = L.r + (color ? half : 0);
    const int hsz = (L.nx * L.ny * (L.sig_hi - L.sig_lo)) >> 1;
    const int oy0 = L.ny > 1 ? (wrap_p(j, L.ny) - j) * hx : 0;
    const int oy1 = L.ny > 1 ? (wrap_m(j, L.ny) - j) * hx : 0;
    const bool upd = UPD && a.fold;
    const double FX_AS(1) *phi_in = nullptr;
    double FX_AS(1) *phi_out = nullptr;
    const int FX_AS(1) *pflags = asp<1>(a.pflags);
    if (upd) {
        const GState *s = st;
        const size_t off = (size_t)a.kb * a.nx * a.ny;
        phi_in = asp<1>(a.phi[cyc_src(s)]) + off;
        phi_out = asp<1>(a.phi[cyc_dst(s)]) + off;
    }
    T out[ZT];
    T rr[ZT], sg[ZT], ex0[ZT], ex1[ZT], ey0[ZT], ey1[ZT], ez0[ZT], ez1[ZT];
    dpair ph[ZT];
    double lim[ZT];
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = min(tt.tz * ZT + z, L.nz - 1);
        const int row = k * plane + j * hx;
        const int q = row + m;
        const bool hs = k >= L.sig_lo && k < L.sig_hi;
        rr[z] = rs[q];
        sg[z] = L.sig[hs ? (color ? hsz : 0) + (k - L.sig_lo) * plane + j * hx + m : 0];
        if (!ZI) {
            const int i = 2 * m + ((color + j + k) & 1);
            const int ip = i + 1 == L.nx ? 0 : i + 1, im = i == 0 ? L.nx - 1 : i - 1;
            ex0[z] = eo[row + (ip >> 1)];
            ex1[z] = eo[row + (im >> 1)];
            ey0[z] = eo[q + oy0];
            ey1[z] = eo[q + oy1];
            ez0[z] = eo[k > 0 ? q - plane : q];
            ez1[z] = eo[k < L.nz - 1 ? q + plane : q];
        }
        if (upd) {
            ph[z] = *(const dpair FX_AS(1) *)(phi_in + (size_t)k * L.nx * L.ny + (size_t)j * L.nx + 2 * m);
            lim[z] = (pflags[k] & PF_SC) ? a.dmax : 1e300;
        }
    }
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = min(tt.tz * ZT + z, L.nz - 1);
        const bool hs = k >= L.sig_lo && k < L.sig_hi;
        T acc = 0;
        if (!ZI) acc = rb_nb_sum(L, k, ex0[z], ex1[z], ey0[z], ey1[z], ez0[z], ez1[z]);
        out[z] = gs_value(rr[z] + acc, L.dg[k] + (hs ? sg[z] : T(0)));
    }
    // Stores outside branches: a lane past the row end works on cell (0, 0) and a slot past
    // the top on plane nz - 1, from the same inputs as the lane owning that cell, so its store
    // repeats the owner's bits.  (A store under a branch made the next plane's arithmetic
    // wait for it to complete.)
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = min(tt.tz * ZT + z, L.nz - 1);
        es[k * plane + j * hx + m] = out[z];
        if (upd) {
            // the pair's red cell is this black cell's x - 1 (black at 2m + 1) or x + 1
            // neighbour (black at 2m), already read as ex1 / ex0
            const bool odd = ((color + j + k) & 1) != 0;
            const double db = fmin(fmax((double)out[z], -lim[z]), lim[z]);
            const double dr = fmin(fmax((double)(odd ? ex1[z] : ex0[z]), -lim[z]), lim[z]);
            dpair o;
            o.x = ph[z].x + (odd ? dr : db);
            o.y = ph[z].y + (odd ? db : dr);
            *(dpair FX_AS(1) *)(phi_out + (size_t)k * L.nx * L.ny + (size_t)j * L.nx + 2 * m) = o;
        }
    }
}

template <typename T, int ZT>
__device__ __forceinline__ void smooth_nat_body(const Lv<T, 1> &L, int t, int color, int zero_init, int lbx) {
    const T3 tt = split3r(t, L.nx, L.ny, lbx);
    const int i = (tt.tx << lbx) + (threadIdx.x & ((1 << lbx) - 1));
    const int j = (tt.ty << (8 - lbx)) + (threadIdx.x >> lbx);
    if (i >= L.nx || j >= L.ny) return;
    for (int z = 0; z < ZT; ++z) {
        const int k = tt.tz * ZT + z;
        if (k >= L.nz) break;
        if (nat_color(L, i, j, k) != color) {
            if (zero_init) L.e[cidx(L, i, j, k)] = T(0);
            continue;
        }
        gs_cell(L, i, j, k, zero_init);
    }
}

// Zero-start pair on a red/black level: the first red half-sweep of a cycle
// (the correction starts at zero, so a red value is r / diag) and the black
// half-sweep after it, in one launch.  A thread per black cell forms the six red
// neighbour values itself, exactly as the red sweep computes them, and also
// stores the red cell of its own (2m, 2m+1) pair, which is one of its two x
// neighbours: the pairs tile each row, so every red cell is written once, with
// the value the red launch would have written.
template <typename T, int ZT>
__device__ __forceinline__ void smooth_zpair_body(const Lv<T, 1> &L, int t, int lbx) {
    const int hx = L.nx >> 1;
    const T3 tt = split3r(t, hx, L.ny, lbx);
    const int m = (tt.tx << lbx) + (threadIdx.x & ((1 << lbx) - 1));
    const int j = (tt.ty << (8 - lbx)) + (threadIdx.x >> lbx);
    if (m >= hx || j >= L.ny) return;
    const int half = (L.nx * L.ny * L.nz) >> 1;
    const int plane = L.ny * hx;
    const int hsz = (L.nx * L.ny * (L.sig_hi - L.sig_lo)) >> 1;
    T FX_AS(1) *e_red = L.e;
    T FX_AS(1) *e_blk = L.e + half;
    const T FX_AS(1) *r_red = L.r, *r_blk = L.r + half;
    const int oy0 = L.ny > 1 ? (wrap_p(j, L.ny) - j) * hx : 0;
    const int oy1 = L.ny > 1 ? (wrap_m(j, L.ny) - j) * hx : 0;
    // red value at red index c of plane kk after a zero-start red half-sweep
    auto red = [&](int c, int kk) {
        const bool hs = kk >= L.sig_lo && kk < L.sig_hi;
        const T sg = L.sig[hs ? (kk - L.sig_lo) * plane + (c - kk * plane) : 0];
        return gs_value(r_red[c] + T(0), L.dg[kk] + (hs ? sg : T(0)));
    };
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = tt.tz * ZT + z;
        if (k >= L.nz) break;
        const int row = k * plane + j * hx;
        const int q = row + m;
        const int i = 2 * m + ((1 + j + k) & 1);
        const int ip = i + 1 == L.nx ? 0 : i + 1, im = i == 0 ? L.nx - 1 : i - 1;
        const bool hs = k >= L.sig_lo && k < L.sig_hi;
        const T rb = r_blk[q];
        const T sb = L.sig[hs ? hsz + (k - L.sig_lo) * plane + j * hx + m : 0];
        const T ex0 = red(row + (ip >> 1), k), ex1 = red(row + (im >> 1), k);
        const T ey0 = red(q + oy0, k), ey1 = red(q + oy1, k);
        const T ez0 = k > 0 ? red(q - plane, k - 1) : red(q, k);
        const T ez1 = k < L.nz - 1 ? red(q + plane, k + 1) : red(q, k);
        const T acc = rb_nb_sum(L, k, ex0, ex1, ey0, ey1, ez0, ez1);
        e_blk[q] = gs_value(rb + acc, L.dg[k] + (hs ? sb : T(0)));
        e_red[q] = (i & 1) ? ex1 : ex0;                  // the pair's red cell: x - 1 or x + 1
    }
}

template <typename T, int ZT>
__global__ __launch_bounds__(256) void k_smooth_zpair(const Inst<T> *I, Work w, int level, int lbx) {
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const int done = wstate(w, b.inst)->done;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    const Lv<T, 1> L = gview(a.lv[level]);
    if (!L.rb) return;                               // the host fuses only all-red/black levels
    smooth_zpair_body<T, ZT>(L, b.t, lbx);
}

// probe (instrumentation): the first tile of each instance that works adds
// the launch's algorithmic bytes for that instance -- one touch each of this
// colour's r, sigma and e, the other colour's e (not read when zero_init),
// and the phi pair read and written where the update is folded in.
template <typename T, int ZI, int ZT, int UPD>
__device__ __forceinline__ void smooth_kernel(const Inst<T> *I, const Work &w, int level, int color, int lbx,
                                              double *probe, int skip_light) {
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const GState *st = wstate(w, b.inst);
    // one exit test with no short-circuit, so that the state's fields and the
    // launch's arguments are read in one round trip (a block past the table's end
    // reads instance 0's; level < 0 never holds)
    const int done = st->done, light = st->light;
    if (!b.ok | (done != 0) | ((skip_light != 0) & (light != 0)) | (level < 0)) return;
    const Lv<T, 1> L = gview(a.lv[level]);
    if (L.rb) {
        if (color > 1) return;
        smooth_rb_body<T, ZI, ZT, UPD>(a, st, L, b.t, color, lbx);
    } else {
        smooth_nat_body<T, ZT>(L, b.t, color, ZI, lbx);
    }
    // after the sweep: an atomic ahead of it would stop the per-plane tables
    // from being read through the scalar cache
    if (probe && b.t == 0 && threadIdx.x == 0 && (L.rb ? color < 2 : true)) {
        const double n = (double)L.nx * L.ny * L.nz, ns = (double)L.nx * L.ny * (L.sig_hi - L.sig_lo);
        double by = sizeof(T) * (0.5 * n + 0.5 * ns + 0.5 * n);
        if (!ZI) by += sizeof(T) * 0.5 * n;
        if (UPD && a.fold && L.rb) by += 16.0 * n;
        atomicAdd(probe, by);
    }
}

// Two register budgets: the compiler's own, and one that keeps at least 8
// waves per SIMD resident (64 VGPRs); the autotuner picks per level.
template <typename T, int ZI, int ZT, int UPD>
__global__ __launch_bounds__(256) void k_smooth(const Inst<T> *I, Work w, int level, int color, int lbx,
                                                double *probe, int skip_light) {
    smooth_kernel<T, ZI, ZT, UPD>(I, w, level, color, lbx, probe, skip_light);
}

template <typename T, int ZI, int ZT, int UPD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_smooth_w8(
    const Inst<T> *I, Work w, int level, int color, int lbx, double *probe, int skip_light) {
    smooth_kernel<T, ZI, ZT, UPD>(I, w, level, color, lbx, probe, skip_light);
}

template <typename T>
__global__ __launch_bounds__(256) void k_restrict(const Inst<T> *I, Work w, int level) {
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const int done = wstate(w, b.inst)->done;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    const Lv<T, 1> C = gview(a.lv[level + 1]);
    const T3 t = split3(b.t, C.nx, C.ny);
    const int I0 = t.tx * BX + threadIdx.x;
    const int J0 = t.ty * BY + threadIdx.y;
    if (I0 >= C.nx || J0 >= C.ny) return;
    const Lv<T, 1> F = gview(a.lv[level]);
    const Xv<T> X = xview(a.xf[level]);
    if (F.rb && X.xy == 1) restrict_cell_rbxy(F, C, X, I0, J0, t.tz);
    else restrict_cell(F, C, X, I0, J0, t.tz);
}

// A thread per column of kProZ planes (black cells only on a red/black
// level): every correction is formed, and every corrected cell read, before
// any cell is updated, so the column's loads are all in flight together.
template <int XY, typename T>
__device__ __forceinline__ void prolong_column(const Lv<T, 1> &F, const Lv<T, 1> &C, const Xv<T> &X, int m, int j,
                                               int k0) {
    T v[kProZ], e[kProZ];
    int c[kProZ];
#pragma unroll
    for (int z = 0; z < kProZ; ++z) {
        const int k = min(k0 + z, F.nz - 1);
        const int i = F.rb ? 2 * m + ((1 + j + k) & 1) : m;
        v[z] = prolong_value<XY>(C, X, i, j, k);
        c[z] = cidx(F, i, j, k);
        e[z] = F.e[c[z]];          // read before any store: a store could alias it
    }
#pragma unroll
    for (int z = 0; z < kProZ; ++z)
        if (k0 + z < F.nz) F.e[c[z]] = e[z] + v[z];
}

// Prolongation fused with the red half-sweep after it, on a red/black level:
// the correction touches only black cells, and the black half-sweep that
// follows recomputes every black cell without reading it, so the corrected
// black values are needed by this red half-sweep alone.  A thread per red cell
// corrects its six black neighbours in registers (same operands, same order as
// prolong_column) and updates itself from them (same expression as the red
// half-sweep); nothing but the red cells is stored.
template <int XY, typename T, int ZT>
__device__ __forceinline__ void prolong_red_body(const Lv<T, 1> &F, const Lv<T, 1> &C, const Xv<T> &X, int t,
                                                 int lbx) {
    const int hx = F.nx >> 1;
    const T3 tt = split3r(t, hx, F.ny, lbx);
    const int m = (tt.tx << lbx) + (threadIdx.x & ((1 << lbx) - 1));
    const int j = (tt.ty << (8 - lbx)) + (threadIdx.x >> lbx);
    if (m >= hx || j >= F.ny) return;
    const int half = (F.nx * F.ny * F.nz) >> 1;
    const int plane = F.ny * hx;
    const T FX_AS(1) *eb = F.e + half;                 // black values before the correction
    T FX_AS(1) *er = F.e;
    const int jp = wrap_p(j, F.ny), jm = wrap_m(j, F.ny);
    const int oy0 = (jp - j) * hx, oy1 = (jm - j) * hx;
    // corrected black value at black index c, fine cell (i, jj, kk)
    auto blk = [&](int c, int i, int jj, int kk) { return eb[c] + prolong_value<XY>(C, X, i, jj, kk); };
#pragma unroll
    for (int z = 0; z < ZT; ++z) {
        const int k = tt.tz * ZT + z;
        if (k >= F.nz) break;
        const int row = k * plane + j * hx;
        const int q = row + m;
        const int i = 2 * m + ((j + k) & 1);
        const int ip = i + 1 == F.nx ? 0 : i + 1, im = i == 0 ? F.nx - 1 : i - 1;
        const bool hs = k >= F.sig_lo && k < F.sig_hi;
        const T rr = F.r[q];
        const T sg = F.sig[hs ? (k - F.sig_lo) * plane + j * hx + m : 0];
        const T ex0 = blk(row + (ip >> 1), ip, j, k), ex1 = blk(row + (im >> 1), im, j, k);
        // one row (ny = 1): the y terms carry a zero coefficient and read the
        // pair's black cell, as the red half-sweep does
        const T ey0 = F.ny > 1 ? blk(q + oy0, i, jp, k) : blk(q, i ^ 1, j, k);
        const T ey1 = F.ny > 1 ? blk(q + oy1, i, jm, k) : blk(q, i ^ 1, j, k);
        const T ez0 = k > 0 ? blk(q - plane, i, j, k - 1) : blk(q, i ^ 1, j, k);
        const T ez1 = k < F.nz - 1 ? blk(q + plane, i, j, k + 1) : blk(q, i ^ 1, j, k);
        const T acc = rb_nb_sum(F, k, ex0, ex1, ey0, ey1, ez0, ez1);
        er[q] = gs_value(rr + acc, F.dg[k] + (hs ? sg : T(0)));
    }
}

template <typename T, int ZT>
__global__ __launch_bounds__(256) void k_prolong_red(const Inst<T> *I, Work w, int level, int lbx) {
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const int done = wstate(w, b.inst)->done;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    const Lv<T, 1> F = gview(a.lv[level]);
    if (!F.rb) return;                               // the host fuses only all-red/black levels
    const Lv<T, 1> C = gview(a.lv[level + 1]);
    const Xv<T> X = xview(a.xf[level]);
    if (X.xy == 1) prolong_red_body<1, T, ZT>(F, C, X, b.t, lbx);
    else if (X.xy == 2) prolong_red_body<2, T, ZT>(F, C, X, b.t, lbx);
    else prolong_red_body<0, T, ZT>(F, C, X, b.t, lbx);
}

// Prolongation into a red/black level halved in x and y and paired in z, a thread
// per coarse column of cz planes.  For each coarse plane the thread loads the
// 3 x 3 neighbourhood of its column once and forms the bilinear values at its four
// child columns; every fine plane of its children then combines the values of its
// parent plane and of the neighbour plane named by the z tables, kept in registers
// as the thread marches up.  Each value goes through lint_xy and lint_z with the
// operands of prolong_value, so the corrections are those of prolong_column bit for
// bit; only black children are corrected (the red ones are overwritten by the next
// red half-sweep without being read).
template <typename T>
__device__ __forceinline__ void prolong_cc_interp(const Lv<T, 1> &C, int K, int Im, int I, int Ip, int Jm, int J,
                                                  int Jp, T (&s)[2][2]) {
    const int ii[3] = {Im, I, Ip}, jj[3] = {Jm, J, Jp};
    T v[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a) v[b][a] = C.e[cidx(C, ii[a], jj[b], K)];
    const T wx[2] = {T(0.75), T(0.25)}, wy[2] = {T(0.75), T(0.25)};
    T w[2][2];
#pragma unroll
    for (int yy = 0; yy < 2; ++yy)
#pragma unroll
        for (int xx = 0; xx < 2; ++xx) w[yy][xx] = wx[xx] * wy[yy];
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
            const int ix[2] = {1, dx ? 2 : 0}, jy[2] = {1, dy ? 2 : 0};
            T u[2][2];
#pragma unroll
            for (int yy = 0; yy < 2; ++yy)
#pragma unroll
                for (int xx = 0; xx < 2; ++xx) u[yy][xx] = v[jy[yy]][ix[xx]];
            s[dy][dx] = lint_xy<2, 2>(w, u);
        }
}

template <typename T>
__global__ __launch_bounds__(256) void k_prolong_cc(const Inst<T> *Ia, Work w, int level, int cz) {
    const Blk b = find_block(w);
    const Inst<T> &a = Ia[b.inst];
    const int done = wstate(w, b.inst)->done;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    const Lv<T, 1> C = gview(a.lv[level + 1]);
    const T3 t = split3(b.t, C.nx, C.ny);
    const int I = t.tx * BX + threadIdx.x;
    const int J = t.ty * BY + threadIdx.y;
    if (I >= C.nx || J >= C.ny) return;
    const Lv<T, 1> F = gview(a.lv[level]);
    const Xv<T> X = xview(a.xf[level]);
    const int Im = wrap_m(I, C.nx), Ip = wrap_p(I, C.nx), Jm = wrap_m(J, C.ny), Jp = wrap_p(J, C.ny);
    const int K0 = t.tz * cz, K1 = min(K0 + cz, C.nz);
    T sp[2][2], sc[2][2], sn[2][2];
    prolong_cc_interp(C, K0 > 0 ? K0 - 1 : K0, Im, I, Ip, Jm, J, Jp, sp);
    prolong_cc_interp(C, K0, Im, I, Ip, Jm, J, Jp, sc);
    for (int K = K0; K < K1; ++K) {
        prolong_cc_interp(C, K + 1 < C.nz ? K + 1 : K, Im, I, Ip, Jm, J, Jp, sn);
        int c[4];
        T e[4], v[4];
        int nf = 0;
#pragma unroll
        for (int dz = 0; dz < 2; ++dz) {
            const int k = 2 * K + dz;
            if (k >= F.nz) break;
            const int kb = X.pkb[k];
            const T wa = X.pwa[k], wb = kb >= 0 ? X.pwb[k] : T(0);
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
                // the black child of this row on plane k: (dx + dy + k) odd
                const int dx = (1 + dy + k) & 1;
                const T s0 = sc[dy][dx];
                const T s1 = kb < 0 ? s0 : (kb < K ? sp[dy][dx] : sn[dy][dx]);
                const T val = lint_z(wa, s0, wb, s1);
                const int q = 2 * dz + dy;
                c[q] = cidx(F, 2 * I + dx, 2 * J + dy, k);
                e[q] = F.e[c[q]];
                v[q] = val;
            }
            nf = 2 * dz + 2;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q < nf) F.e[c[q]] = e[q] + v[q];
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                sp[dy][dx] = sc[dy][dx];
                sc[dy][dx] = sn[dy][dx];
            }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_prolong(const Inst<T> *I, Work w, int level) {
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const int done = wstate(w, b.inst)->done;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    const Lv<T, 1> F = gview(a.lv[level]);
    const int nxe = F.rb ? F.nx >> 1 : F.nx;      // black cells per row on a red/black level
    const T3 t = split3(b.t, nxe, F.ny);
    const int m = t.tx * BX + threadIdx.x;
    const int j = t.ty * BY + threadIdx.y;
    if (m >= nxe || j >= F.ny) return;
    const Lv<T, 1> C = gview(a.lv[level + 1]);
    const Xv<T> X = xview(a.xf[level]);
    if (X.xy == 1) prolong_column<1>(F, C, X, m, j, t.tz * kProZ);
    else if (X.xy == 2) prolong_column<2>(F, C, X, m, j, t.tz * kProZ);
    else prolong_column<0>(F, C, X, m, j, t.tz * kProZ);
}

// ------------------------------------------------------------- temporal blocking
// On a red/black level small enough for its launches to be latency-bound, the pre-smoothing
// sweeps and the restriction are one launch, and so are the prolongation and the post-smoothing
// sweeps.  A block owns a tile of kTbT x kTbT columns of every plane and keeps a box of the
// tile plus a kTbH-cell ring of e in LDS.  Each half-sweep over the box leaves one ring
// fewer valid, so nu sweeps need a ring of 2 nu cells (nu <= 2 here), recomputed by every block
// that needs it.  Every value goes through the expressions of the launches it replaces (the
// zero-start value, nb6, gs_value and res_value; the lateral and z interpolants of prolong_value;
// the restriction's sums in order; the clipped Newton update) with the same operands, so the
// results are theirs bit for bit.
//   pre:  nu zero-start sweeps on e (red then black), the restriction of the red children's
//         residuals and of sigma into the coarse level, and the tile's black values
//         stored in ealt (the only ones the post launch reads);
//   post: black values of ealt plus the interpolated correction, nu sweeps (the first red
//         half-sweep reads the corrected black values, as the fused prolongation does),
//         and both colours of the tile stored in e, or on the finest level phi_out =
//         phi_in + clip(e) (nothing reads e there).
// The post launch reads ealt around its tile while other blocks store e, so the two must not
// overlap: ealt is an array of the level, the finer level's red half (dead between that
// level's restriction and its next red half-sweep), or, on the finest level, e's own
// black half (no e is stored there).
//
// What bounds it: four phases of LDS reads, each a chain of latencies (about 0.5 us), and the
// LDS bandwidth of the box (4 times the tile's cells) on levels with many planes.  A wave
// holds 64 box columns of one (x + y) parity, so the planes of its cells of one colour are the
// same for all its lanes: the per-plane coefficients sit in scalar registers, the colours lie
// in LDS arrays of their own (a column's cell and its x neighbours share or adjoin a pair), and
// a wave's reads are contiguous.  Right-hand sides and reciprocal diagonals stay in registers
// over all sweeps.  ZQ, the cells of one colour per thread, follows the level's planes.
// Extents need not be multiples of the tile: the last tiles own what is left.
constexpr int kTbThreads = kTbShares * kTbW * kTbW;
constexpr int kTbPl = kTbW * kTbW / 2;        // box cells of one colour per plane
constexpr int kTbCW = kTbW / 2 + 2;           // coarse columns under a box, with the interpolation's neighbours
static_assert(kTbW == 16, "a wave's 64 lanes are 8 rows of 8 pairs");

struct TbCol {
    int gi, gj, q0;                        // global column, its pair index in a plane
    int bx, by, tx, ty;                    // box column, tile
    int ring;                              // 0 inside the tile
    int li, xo;                            // LDS pair index in a plane; offset of the x neighbours' other pair
    int par, z0, zf;                       // (x + y) parity, first cell index of the share, first one
                                           // no earlier share has (uniform in a wave)
    int np;                                // planes of one colour's array, two pads included
    bool own;                              // column of the tile and of the grid
};

template <int ZQ, typename V>
__device__ __forceinline__ TbCol tb_col(const V &L, int t) {
    const int ntx = (L.nx + kTbT - 1) / kTbT;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    TbCol c;
    c.ty = t / ntx;
    c.tx = t - c.ty * ntx;
    c.par = wave & 1;
    // shares of ZQ cells; the last ones move down so that none reaches past the top (cells of
    // two shares get the same value twice)
    const int nc = (L.nz + 1) / 2;
    c.zf = (wave >> 2) * ZQ;
    c.z0 = max(0, min(c.zf, nc - ZQ));
    c.np = max(L.nz, 2 * ZQ) + 2;
    c.by = (lane >> 3) + 8 * ((wave >> 1) & 1);
    c.bx = 2 * (lane & 7) + ((c.by + c.par) & 1);
    int gi = c.tx * kTbT - kTbH + c.bx, gj = c.ty * kTbT - kTbH + c.by;
    const int rx = c.bx < kTbH ? kTbH - c.bx : (c.bx >= kTbH + kTbT ? c.bx - (kTbH + kTbT - 1) : 0);
    const int ry = c.by < kTbH ? kTbH - c.by : (c.by >= kTbH + kTbT ? c.by - (kTbH + kTbT - 1) : 0);
    c.ring = rx > ry ? rx : ry;
    c.own = c.ring == 0 && gi < L.nx && gj < L.ny;
    gi += gi < 0 ? L.nx : (gi >= L.nx ? -L.nx : 0);
    gj += gj < 0 ? L.ny : (gj >= L.ny ? -L.ny : 0);
    c.gi = gi;
    c.gj = gj;
    c.q0 = gj * (L.nx >> 1) + (gi >> 1);
    c.li = c.by * (kTbW / 2) + (c.bx >> 1);
    c.xo = (c.bx & 1) ? 1 : -1;
    return c;
}

// Colour col's array of the box (the caller's column added): plane k at k kTbPl.  The planes
// below the lowest and above the highest cell are pads of zeros, so that every cell reads both
// z neighbours (with weight 0 at the contacts) at fixed offsets.
template <typename T>
__device__ __forceinline__ T FX_AS(3) *tb_array(T FX_AS(3) *box, const TbCol &c, int col) {
    return box + (col * c.np + 1) * kTbPl + c.li;
}
template <typename T>
__device__ __forceinline__ void tb_pads(T FX_AS(3) *box, const TbCol &c, int nz) {
    const int t = threadIdx.x;
    if (t < 4 * kTbPl) box[((t >> 8) * c.np + ((t >> 7) & 1) * (nz + 1)) * kTbPl + (t & (kTbPl - 1))] = T(0);
}

// Plane of this thread's z-th cell of colour col (past the top on levels with few planes or an
// odd count: such cells are formed from whatever lies there and never stored).
__device__ __forceinline__ int tb_k(const TbCol &c, int col, int z) { return 2 * (c.z0 + z) + ((col + c.par) & 1); }

// This thread's cells of both colours: right-hand sides and reciprocal diagonals (vectors),
// coefficients (scalars).
template <typename T, int ZQ>
struct TbCells {
    T r[2][ZQ], iv[2][ZQ], cx[2][ZQ], cm[2][ZQ], cp[2][ZQ];

    // idg: room for the reciprocal diagonals of the planes without sigma, formed once per block
    // (a division per cell cost 3 us a launch); stores: LDS stores of the caller to be published
    // by the same barrier, after this thread's loads have been issued.
    template <typename F>
    __device__ __forceinline__ void load(const Lv<T, 1> &L, const TbCol &c, T FX_AS(3) *idg, F stores) {
        const int plane = L.ny * (L.nx >> 1), half = plane * L.nz, hsz = plane * (L.sig_hi - L.sig_lo);
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int z = 0; z < ZQ; ++z) {
                const int k = min(tb_k(c, col, z), L.nz - 1);
                r[col][z] = L.r[col * half + k * plane + c.q0];
                iv[col][z] = T(0);
                if (has_sig(L, k)) iv[col][z] = L.sig[col * hsz + (k - L.sig_lo) * plane + c.q0];
            }
        for (int k = threadIdx.x; k < L.nz; k += kTbThreads) idg[k] = T(1) / L.dg[k];
        stores();
        __syncthreads();
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int z = 0; z < ZQ; ++z) {
                const int k = min(tb_k(c, col, z), L.nz - 1);
                cx[col][z] = L.cxy[k];
                cm[col][z] = k > 0 ? L.czm[k] : T(0);
                cp[col][z] = k < L.nz - 1 ? L.czp[k] : T(0);
                if (has_sig(L, k)) iv[col][z] = T(1) / (L.dg[k] + iv[col][z]);
                else iv[col][z] = idg[k];
            }
    }
    // neighbour sum of colour col's z-th cell; eo: the other colour's array
    __device__ __forceinline__ T nb(const TbCol &c, const T FX_AS(3) *eo, int col, int z) const {
        const T FX_AS(3) *e = eo + (2 * c.z0 + ((col + c.par) & 1)) * kTbPl + 2 * z * kTbPl;
        return nb6(cx[col][z], cx[col][z], cm[col][z], cp[col][z], e[0], e[c.xo], e[kTbW / 2], e[-(kTbW / 2)], e[-kTbPl],
                   e[kTbPl]);
    }
    // One half-sweep of colour col over the box columns within ring R (ZI: from a zero
    // start).  Cells of one colour are not neighbours, so the new values of a group of cells
    // are formed before any of them is stored (the group bounds the registers held).
    template <int ZI, int BAR = 1>
    __device__ __forceinline__ void half_sweep(const TbCol &c, int nz, T FX_AS(3) *box, int col, int R) const {
        constexpr int G = ZQ <= 4 ? ZQ : ZQ / 2;
        T FX_AS(3) *es = tb_array(box, c, col);
        const T FX_AS(3) *eo = tb_array(box, c, 1 - col);
        if (c.ring <= R) {
#pragma unroll
            for (int z0 = 0; z0 < ZQ; z0 += G) {
                T v[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int z = z0 + g;
                    v[g] = (ZI ? r[col][z] : r[col][z] + nb(c, eo, col, z)) * iv[col][z];
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int k = tb_k(c, col, z0 + g);
                    if (k < nz) es[k * kTbPl] = v[g];
                }
            }
        }
        if (BAR) __syncthreads();
    }
};

template <typename T, int ZQ>
__global__ __launch_bounds__(kTbThreads) void k_pre_tb(const Inst<T> *I, Work w, int level, int nu) {
    extern __shared__ double tb_raw[];
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const GState *st = wstate(w, b.inst);
    const int done = st->done, light = st->light;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    if (light) nu = 1;                         // the sweeps after the first are left out
    const Lv<T, 1> L = gview(a.lv[level]);
    const Xv<T> X = xview(a.xf[level]);
    const Lv<T, 1> C = gview(a.lv[level + 1]);
    T FX_AS(3) *box = asp<3>((T *)tb_raw);
    const TbCol c = tb_col<ZQ>(L, b.t);
    const int nz = L.nz;
    tb_pads(box, c, nz);
    TbCells<T, ZQ> m;
    m.load(L, c, box + 2 * c.np * kTbPl, [] {});
    // sigma of the tile's coarse cells (kTbT/2 x kTbT/2 columns of every coarse plane)
    constexpr int kC = kTbT / 2;
    for (int u = threadIdx.x; u < kC * kC * (C.sig_hi - C.sig_lo); u += kTbThreads) {
        const int K = C.sig_lo + u / (kC * kC), J = c.ty * kC + u / kC % kC, I0 = c.tx * kC + u % kC;
        if (I0 >= C.nx || J >= C.ny) continue;
        const int ks = X.cks[K], cnt = X.ccnt[K];
        double ss = 0.0;
        for (int dz = 0; dz < cnt; ++dz) {
            const double wz = (double)X.fthick[ks + dz] / (double)X.cthick[K];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const T sg = has_sig(L, ks + dz) ? L.sig[sidx(L, 2 * I0 + (q & 1), 2 * J + (q >> 1), ks + dz)] : T(0);
                ss = fmad(wz, (double)sg, ss);
            }
        }
        C.sig[sidx(C, I0, J, K)] = (T)(ss * 0.25);
    }
    m.template half_sweep<1>(c, nz, box, 0, 2 * nu);
    m.template half_sweep<0>(c, nz, box, 1, 2 * nu - 1);
    if (nu > 1) {
        m.template half_sweep<0>(c, nz, box, 0, 2);
        m.template half_sweep<0>(c, nz, box, 1, 1);
    }
    T FX_AS(3) *red = tb_array(box, c, 0);
    const T FX_AS(3) *blk = tb_array(box, c, 1);
    const int plane = L.ny * (L.nx >> 1);
    if (c.own) {
        // the tile's black values for the post launch; its red residuals into the red cells
        T FX_AS(1) *ealt = asp<1>(a.lv[level].ealt);
#pragma unroll
        for (int z = 0; z < ZQ; ++z) {
            const int k = tb_k(c, 1, z);
            if (k < nz) ealt[k * plane + c.q0] = blk[k * kTbPl];
        }
#pragma unroll
        for (int z = 0; z < ZQ; ++z) {
            const int k = tb_k(c, 0, z);
            if (k >= nz || c.z0 + z < c.zf) continue;
            T d = L.dg[k];
            if (has_sig(L, k)) d += L.sig[(k - L.sig_lo) * plane + c.q0];
            red[k * kTbPl] = res_value(m.r[0][z], d, red[k * kTbPl], m.nb(c, blk, 0, z));
        }
    }
    __syncthreads();
    for (int u = threadIdx.x; u < kC * kC * C.nz; u += kTbThreads) {
        const int K = u / (kC * kC), cj = u / kC % kC, ci = u % kC;
        const int J = c.ty * kC + cj, I0 = c.tx * kC + ci;
        if (I0 >= C.nx || J >= C.ny) continue;
        const int ks = X.cks[K], cnt = X.ccnt[K];
        double sr = 0.0;
        for (int dz = 0; dz < cnt; ++dz) {
            const double wz = (double)X.fthick[ks + dz] / (double)X.cthick[K];
            const T FX_AS(3) *p = box + (ks + dz + 1) * kTbPl + (kTbH + 2 * cj) * (kTbW / 2) + kTbH / 2 + ci;
            sr = fmad(wz, (double)p[0], sr);
            sr = fmad(wz, (double)p[kTbW / 2], sr);
        }
        C.r[cidx(C, I0, J, K)] = (T)(sr * 0.25);
    }
}

template <typename T, int ZQ, int FINEST>
__global__ __launch_bounds__(kTbThreads) void k_post_tb(const Inst<T> *I, Work w, int level, int nu) {
    extern __shared__ double tb_raw[];
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const GState *st = wstate(w, b.inst);
    const int done = st->done, light = st->light;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    if (light) nu = 1;                         // one sweep: the fused prolongation's and the black after it
    const Lv<T, 1> F = gview(a.lv[level]);
    const Lv<T, 1> C = gview(a.lv[level + 1]);
    const Xv<T> X = xview(a.xf[level]);
    T FX_AS(3) *box = asp<3>((T *)tb_raw);
    const TbCol c = tb_col<ZQ>(F, b.t);
    const int nz = F.nz;
    const int plane = F.ny * (F.nx >> 1), half = plane * nz;
    // The coarse values under the box (kTbCW x kTbCW coarse columns, every coarse plane), one
    // load each, above the box in LDS; then this thread's cells.  Box column bx lies over coarse
    // box column (tile x - kTbH + bx) / 2 - (tile x kTbT/2 - kTbH/2 - 1), its x neighbour one
    // further on the side of its parity, as prolong_value takes them (wrapping included).
    T FX_AS(3) *cb = box + 2 * c.np * kTbPl;
    const int cx0 = c.tx * (kTbT / 2) - kTbH / 2 - 1, cy0 = c.ty * (kTbT / 2) - kTbH / 2 - 1;
    constexpr int CU = (kTbCW * kTbCW * ZQ * kTbShares + kTbThreads - 1) / kTbThreads;   // C.nz <= 4 ZQ
    T cv[CU];
#pragma unroll
    for (int q = 0; q < CU; ++q) {
        const int u = min((int)threadIdx.x + q * kTbThreads, kTbCW * kTbCW * C.nz - 1);
        const int K = u / (kTbCW * kTbCW), rem = u - K * kTbCW * kTbCW;
        const int cj = rem / kTbCW, ci = rem - cj * kTbCW;
        int I0 = cx0 + ci, J = cy0 + cj;
        I0 += I0 < 0 ? C.nx : (I0 >= C.nx ? -C.nx : 0);
        J += J < 0 ? C.ny : (J >= C.ny ? -C.ny : 0);
        cv[q] = C.e[cidx(C, I0, J, K)];
    }
    T eb[ZQ];
    const T FX_AS(1) *ea = asp<1>(a.lv[level].ealt);
#pragma unroll
    for (int z = 0; z < ZQ; ++z) eb[z] = ea[min(tb_k(c, 1, z), nz - 1) * plane + c.q0];
    tb_pads(box, c, nz);
    TbCells<T, ZQ> m;
    m.load(F, c, cb + kTbCW * kTbCW * C.nz, [&] {
#pragma unroll
        for (int q = 0; q < CU; ++q) {
            const int u = threadIdx.x + q * kTbThreads;
            if (u < kTbCW * kTbCW * C.nz) cb[u] = cv[q];
        }
    });
    T FX_AS(3) *blk = tb_array(box, c, 1);
    if (c.ring <= 2 * nu) {
        // the correction of the black cells: lint_z of the lateral interpolants on the parent
        // and neighbour planes (prolong_value's weights and operands).  The planes are paired,
        // so cell z's parent is coarse plane z0 + z and its neighbour the next one up (odd
        // planes) or down (even ones, b = 0): ZQ + 1 interpolants serve the share.
        const T wx[2] = {T(0.75), T(0.25)}, wy[2] = {T(0.75), T(0.25)};
        T wgt[2][2];
#pragma unroll
        for (int yy = 0; yy < 2; ++yy)
#pragma unroll
            for (int xx = 0; xx < 2; ++xx) wgt[yy][xx] = wx[xx] * wy[yy];
        const int gu = c.tx * kTbT - kTbH + c.bx, gv = c.ty * kTbT - kTbH + c.by;   // unwrapped
        const int ci = (gu >> 1) - cx0, cj = (gv >> 1) - cy0;
        const int dx = (gu & 1) ? 1 : -1, dy = ((gv & 1) ? 1 : -1) * kTbCW, o = cj * kTbCW + ci;
        const int b1 = (1 + c.par) & 1;
        auto lateral = [&](int q) {
            const int K = max(0, min(c.z0 + q - 1 + b1, C.nz - 1));
            const T FX_AS(3) *p = cb + K * (kTbCW * kTbCW) + o;
            T v[2][2];
            v[0][0] = p[0];
            v[0][1] = p[dx];
            v[1][0] = p[dy];
            v[1][1] = p[dy + dx];
            return lint_xy<2, 2>(wgt, v);
        };
        T lo = lateral(0);
#pragma unroll
        for (int z = 0; z < ZQ; ++z) {
            const T hi = lateral(z + 1);
            const int kk = tb_k(c, 1, z), k = min(kk, nz - 1);
            const int kb = X.pkb[k];
            const T v = eb[z] + lint_z(T(X.pwa[k]), b1 ? lo : hi, kb >= 0 ? T(X.pwb[k]) : T(0), b1 ? hi : lo);
            if (kk < nz) blk[k * kTbPl] = v;
            lo = hi;
        }
    }
    __syncthreads();
    m.template half_sweep<0>(c, nz, box, 0, 2 * nu - 1);
    if (nu > 1) {
        m.template half_sweep<0>(c, nz, box, 1, 2);
        m.template half_sweep<0>(c, nz, box, 0, 1);
    }
    // phi of the tile's cells, in flight during the last half-sweep
    const size_t off = (size_t)a.kb * a.nx * a.ny;
    const int col0 = c.gj * F.nx + c.gi, nxy = F.nx * F.ny;
    double ph[2][ZQ];
    if (FINEST && c.own) {
        const double FX_AS(1) *phi_in = asp<1>(a.phi[cyc_src(st)]) + off;
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int z = 0; z < ZQ; ++z) ph[col][z] = phi_in[(size_t)min(tb_k(c, col, z), nz - 1) * nxy + col0];
    }
    // each thread reads back its own cells alone: no barrier
    m.template half_sweep<0, 0>(c, nz, box, 1, 0);
    if (!c.own) return;
    if (FINEST) {
        double FX_AS(1) *phi_out = asp<1>(a.phi[cyc_dst(st)]) + off;
        const int FX_AS(1) *pflags = asp<1>(a.pflags);
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int z = 0; z < ZQ; ++z) {
                const int k = tb_k(c, col, z);
                if (k >= nz) continue;
                const double lim = (pflags[k] & PF_SC) ? a.dmax : 1e300;
                const double d = (double)tb_array(box, c, col)[k * kTbPl];
                phi_out[(size_t)k * nxy + col0] = ph[col][z] + fmin(fmax(d, -lim), lim);
            }
    } else {
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int z = 0; z < ZQ; ++z) {
                const int k = tb_k(c, col, z);
                if (k < nz) F.e[col * half + k * plane + c.q0] = tb_array(box, c, col)[k * kTbPl];
            }
    }
}

// ------------------------------------------- temporal blocking, marching in z
// The same two launches on levels too large for boxes of whole columns: a block owns a
// kZmT x kZmT tile of a chunk of planes, with a ring of kZmH cells in x and y and kZmH planes at
// either end, and marches up in z with all half-sweeps in flight: in step k the first one works on
// plane k, each later stage one plane below the stage before it, and the last (the residual,
// or the finished values) on plane k - 4.  A thread owns a storage pair (a red and a black
// cell of one row) through the march, so a cell's z neighbours and its x neighbour in the pair
// are the thread's own recent values of the other colour, in registers; the other x neighbour
// and the two y neighbours come from the stage's plane in LDS, double-buffered, one barrier
// per step.  Right-hand sides and sigma are loaded two planes ahead, once per block.
// Expressions and operands are those of the half-sweep launches (nb6, gs_value's product,
// res_value, lint_xy, lint_z, the restriction's sums in order): the same bits.  Invalid values
// at the ring and beyond a chunk's ends move inwards one cell per stage and never reach the
// tile.  A light cycle passes the last two half-sweeps' values through.
//
// What bounds it: on 256 x 256 x 120 cells the half-sweep launches and transfers of a cycle read
// and write 1.2 GB (231 us); here r, sigma, phi and the black values are read once per launch
// (0.59 GB with the rings, FP32 0.37, by counters), and the latency of a step's chain of LDS reads,
// FP64 operations and barrier over 1.56 x (zl + 8) / zl cell updates takes over: 77 + 82 us
// (FP32 65 + 60, launches 138; 32 instances of 64 x 64 x 24: 29 + 35, launches 141).  Tiles of
// 32 x 16 with two blocks per compute unit measured 82 + 87, 68 + 64 and 27 + 34; an order of the
// tiles that shares more of the rings in L2 fetched 15% less in the same time.  The form without
// spaced waits and scalar extents took 71 + 78, FP32 57 + 56, and 29 + 37 on the 32 instances.
constexpr int kZmThreads = 832;               // 800 pairs of the box, whole waves
constexpr int kZmP = (kZmT + 2 * kZmH) / 2;   // pairs per box row
constexpr int kZmN = kZmP * (kZmT + 2 * kZmH);
constexpr int kZmPad = 24;                    // LDS neighbours of the box's edge cells stay inside
constexpr int kZmA = kZmN + 2 * kZmPad;       // one stage's plane
constexpr int kZmCW = kZmP + 2;               // coarse columns and rows under a box, with neighbours
static_assert(kZmThreads % 64 == 0 && kZmThreads >= kZmN && kZmPad > kZmP, "box");

__device__ __forceinline__ float uniform_value(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uniform_value(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int V> using ic = std::integral_constant<int, V>;

__device__ __forceinline__ int uniform_value(int v) {
    // as asm: the builtin is dropped where the compiler sees the value to be uniform, and what
    // is formed from it stays in vector registers (the nops keep a scalar use at its distance)
    int o;
    asm volatile("s_nop 1\n\tv_readfirstlane_b32 %0, %1\n\ts_nop 4" : "=s"(o) : "v"(v));
    return o;
}
// A level whose extents are known to be the same in all lanes: plane addresses stay scalar.
template <typename A>
__device__ __forceinline__ auto zm_view(const A &a) {
    auto L = gview(a);
    L.nx = uniform_value(L.nx);
    L.ny = uniform_value(L.ny);
    L.nz = uniform_value(L.nz);
    L.sig_lo = uniform_value(L.sig_lo);
    L.sig_hi = uniform_value(L.sig_hi);
    return L;
}
// A loaded value in a register of its own: the next load into the source's register may follow
// at once, where the compiler would else load elsewhere and move that value, waiting for it.
__device__ __forceinline__ float zm_take(float v) {
    float o;
    asm("v_mov_b32 %0, %1" : "=&v"(o) : "v"(v));
    return o;
}
__device__ __forceinline__ double zm_take(double v) {
    double o;
    asm("v_mov_b64 %0, %1" : "=&v"(o) : "v"(v));
    return o;
}
__device__ __forceinline__ dpair zm_take(dpair v) { return dpair{zm_take(v.x), zm_take(v.y)}; }
struct ZmBlk {
    int tx, ty, z0, z1, k0;                // tile, planes [z0, z1) of the chunk, first plane of the march
    int q0;                                // global pair index in a plane
    int lp, x[2];                          // LDS index; of the red cell's other x neighbour on even / odd planes
    int row, m, gi2, gj;                   // box row and pair; wrapped pair column and row
    bool own;                              // pair of the tile and of the grid
};
template <typename V>
__device__ __forceinline__ ZmBlk zm_block(const V &L, int t, int zl) {
    ZmBlk c;
    const int nzc = (L.nz + zl - 1) / zl, ntx = (L.nx + kZmT - 1) / kZmT;
    // the chunks of a tile, then the tiles of a row, on one XCD (divisions leave the scalar unit)
    const int q = t / nzc, zc = uniform_value(t - q * nzc), qy = q / ntx;
    c.tx = uniform_value(q - qy * ntx);
    c.ty = uniform_value(qy);
    c.z0 = zc * zl;
    c.z1 = min(c.z0 + zl, L.nz);
    c.k0 = max(c.z0 - kZmH, 0);
    const int tid = min((int)threadIdx.x, kZmN - 1);
    c.row = tid / kZmP;
    c.m = tid - c.row * kZmP;
    const int hx = L.nx >> 1;
    int gm = c.tx * (kZmT / 2) - kZmH / 2 + c.m, gj = c.ty * kZmT - kZmH + c.row;
    const bool in = c.m >= kZmH / 2 && c.m < kZmH / 2 + kZmT / 2 && c.row >= kZmH && c.row < kZmH + kZmT;
    c.own = in && gm < hx && gj < L.ny && (int)threadIdx.x < kZmN;
    gm = (gm % hx + hx) % hx;              // extents may be smaller than the box
    gj = (gj % L.ny + L.ny) % L.ny;
    c.gi2 = gm;
    c.gj = gj;
    c.q0 = gj * hx + gm;
    c.lp = kZmPad + c.row * kZmP + c.m;
    c.x[0] = c.lp + ((c.row & 1) ? 1 : -1);    // ny even: the box row's parity is the grid row's
    c.x[1] = c.lp + ((c.row & 1) ? -1 : 1);
    return c;
}

// Tables in LDS of the march's planes (zeros past the top, so that what is formed there is 0):
// reciprocal and plain diagonal, coefficients.
template <typename T>
struct ZmTab {
    T FX_AS(3) *p;
    int k0, n;
    __device__ __forceinline__ void fill(const Lv<T, 1> &L) const {
        for (int q = threadIdx.x; q < n; q += kZmThreads) {
            const int k = k0 + q;
            const bool in = k < L.nz;
            const T dg = in ? L.dg[k] : T(0);
            p[5 * q] = in ? T(1) / dg : T(0);
            p[5 * q + 1] = dg;
            p[5 * q + 2] = in ? L.cxy[k] : T(0);
            p[5 * q + 3] = in && k > 0 ? L.czm[k] : T(0);
            p[5 * q + 4] = in && k < L.nz - 1 ? L.czp[k] : T(0);
        }
    }
    __device__ __forceinline__ T at(int k, int q) const { return uniform_value((T)p[5 * (max(k, k0) - k0) + q]); }
};

// Reciprocal diagonals: uniform over a plane without sigma; in a chunk with sigma, the
// thread's own of the last four planes in LDS (each reads back what it wrote: no barrier).
template <typename T, int SIG>
struct ZmIv {
    T FX_AS(3) *p;                         // slots [colour][plane mod 4]
    const T (&uni)[5];                     // the uniform values of planes k .. k - 4
    __device__ __forceinline__ T get(const Lv<T, 1> &L, int col, int k, int d) const {
        if (!SIG) return uni[d];
        return p[(4 * col + ((k - d) & 3)) * kZmN];
    }
    __device__ __forceinline__ void put(int col, int k, T v) const { p[(4 * col + (k & 3)) * kZmN] = v; }
};

// A value of a stage's plane: other colour's neighbours in LDS (x: the x neighbour outside the
// pair), the pair's own cell and the z neighbours in registers.
template <typename T>
__device__ __forceinline__ T zm_nb(const T FX_AS(3) *pl, const ZmBlk &c, int x, T cx, T cm, T cp, T pair, T lo, T hi) {
    return nb6(cx, cx, cm, cp, pair, pl[x], pl[c.lp + kZmP], pl[c.lp - kZmP], lo, hi);
}
// gs_value with the reciprocal at hand
template <typename T>
__device__ __forceinline__ T zm_gs(T rhs, T iv) {
#pragma clang fp contract(off)
    return rhs * iv;
}
// The stages' planes below the first one: finite values, which zero coefficients then drop.
template <typename T>
__device__ __forceinline__ void zm_clear(T FX_AS(3) *lds, int n) {
    for (int u = threadIdx.x; u < n; u += kZmThreads) lds[u] = T(0);
}
template <int N, typename T>
__device__ __forceinline__ void zm_push(T (&h)[N], T v) {
#pragma unroll
    for (int q = N - 1; q > 0; --q) h[q] = h[q - 1];
    h[0] = v;
}

// Keeps the scheduler from gathering the loads of all stages, which FP64 has no registers for.
template <typename T, int SIG>
__device__ __forceinline__ void zm_fence() {
    if (sizeof(T) == 8 && SIG) __builtin_amdgcn_sched_barrier(0);
}

// The operands of a plane, loaded two steps ahead; o, os: the pair's cell index on the plane and
// in sigma's planes (past the top: the last plane's; without sigma: the nearest's, unused).
// The indices go up plane by plane: a product per load cost more than the addition.
template <typename V>
__device__ __forceinline__ int zm_next(const V &L, int k, int plane) { return k + 1 < L.nz ? plane : 0; }
template <typename V>
__device__ __forceinline__ int zm_next_sig(const V &L, int k, int plane) {
    return k + 1 > L.sig_lo && k + 1 < L.sig_hi ? plane : 0;
}
template <typename V>
__device__ __forceinline__ int zm_first_sig(const V &L, int k, int plane) {
    return max(0, min(k, L.sig_hi - 1) - L.sig_lo) * plane;
}
template <typename T>
struct ZmIn {
    T r0, r1, s0, s1;
    template <int SIG>
    __device__ __forceinline__ ZmIn take() const {
        return {zm_take(r0), zm_take(r1), SIG ? zm_take(s0) : T(0), SIG ? zm_take(s1) : T(0)};
    }
    template <int SIG>
    __device__ __forceinline__ void load(const Lv<T, 1> &L, int o, int os, int half, int half_s) {
        r0 = L.r[o];
        r1 = L.r[half + o];
        s0 = s1 = T(0);
        if (SIG) {
            s0 = L.sig[os];
            s1 = L.sig[half_s + os];
        }
    }
};
// The march, in pairs of steps; sigma's code only in the chunks whose planes meet sigma.
template <typename V>
__device__ __forceinline__ bool zm_sig(const V &L, int k0, int k1) {
    return k0 < L.sig_hi && k1 > L.sig_lo && L.sig_hi > L.sig_lo;
}
template <typename V, typename S>
__device__ __forceinline__ void zm_march(const V &L, int k0, int k1, S &&step) {
    if (zm_sig(L, k0, k1)) {
#pragma unroll 1
        for (int k = k0; k < k1; k += 2) {
            step(k, 0, ic<1>());
            step(k + 1, 1, ic<1>());
        }
    } else {
#pragma unroll 1
        for (int k = k0; k < k1; k += 2) {
            step(k, 0, ic<0>());
            step(k + 1, 1, ic<0>());
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kZmThreads) void k_pre_zm(const Inst<T> *I, Work w, int level, int nu, int zl) {
    extern __shared__ double tb_raw[];
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const GState *st = wstate(w, b.inst);
    const int done = st->done, light = st->light;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    const bool two = nu > 1 && !light;              // the second sweep is made
    const Lv<T, 1> L = zm_view(a.lv[level]), C = gview(a.lv[level + 1]);
    const Xv<T> X = xview(a.xf[level]);
    const ZmBlk c = zm_block(L, b.t, zl);
    const int k1 = c.z1 + kZmH + 1;                 // the last plane's odd rows follow a step later
    const int nz = L.nz, plane = (L.nx >> 1) * L.ny, half = plane * nz;
    T FX_AS(1) *ealt = asp<1>(a.lv[level].ealt);
    // LDS: double-buffered planes of the four half-sweeps, the residuals and the pair's sigmas
    T FX_AS(3) *lds = asp<3>((T *)tb_raw);
    auto buf = [&](int stage, int par) { return lds + (2 * stage + par) * kZmA; };
    T FX_AS(3) *ivp = lds + 14 * kZmA + c.lp - kZmPad;
    const ZmTab<T> tab{lds + 14 * kZmA + 8 * kZmN, c.k0, kZmTab(zl)};
    double FX_AS(3) *wzt = (double FX_AS(3) *)(tab.p + ((5 * kZmTab(zl) + 1) & ~1));
    zm_clear(lds, 14 * kZmA);
    tab.fill(L);
    for (int q = threadIdx.x; q < kZmTab(zl); q += kZmThreads) {
        const int k = c.k0 + q;
        wzt[q] = k < nz ? (double)X.fthick[k] / (double)X.cthick[k >> 1] : 0.0;
    }
    auto wz_of = [&](int k) { return uniform_value((double)wzt[max(k - c.k0, 0)]); };
    T rr[5] = {}, rb[4] = {}, a0[3] = {}, b0[3] = {}, a1[3] = {}, b1[3] = {};
    T cx[5] = {}, cm[5] = {}, cp[5] = {}, idg[5] = {};
    T s4 = T(0);                                           // red sigma of the next residual plane
    double sr = 0.0, ss = 0.0;
    ZmIn<T> in[2];
    // cell indices of the planes loaded next: k + 2 of a step
    const int half_s = plane * (L.sig_hi - L.sig_lo);
    int o = c.k0 * plane + c.q0, os = zm_first_sig(L, c.k0, plane) + c.q0;
    auto advance = [&](int k) {
        o += zm_next(L, k, plane);
        os += zm_next_sig(L, k, plane);
    };
    int os4 = zm_first_sig(L, c.k0 - 3, plane) + c.q0;
    const bool any_sig = zm_sig(L, c.k0, k1);
    for (int q = 0; q < 2; ++q) {
        if (any_sig) in[q].template load<1>(L, o, os, half, half_s);
        else in[q].template load<0>(L, o, os, half, half_s);
        advance(c.k0 + q);
    }
    // the coarse column of this thread's row and the one below it: even rows hold its sums
    const int gI = c.gi2, gJ = c.gj >> 1;
    const bool own_c = c.own && !(c.row & 1);
    // the loads above are waited for here: the march's own waits then count its own loads
    __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0)
    __syncthreads();                                       // tables
    auto step = [&](int k, int cur, auto sig_) {
        constexpr int SIG = decltype(sig_)::value;
        const int prv = cur ^ 1;                           // k0 is even: cur is the plane's parity
        // waits are in the order of issue: what is needed soonest is loaded first
        const T s4c = SIG ? zm_take(s4) : T(0);
        const ZmIn<T> v = in[cur].template take<SIG>();
        if (SIG) {
            s4 = L.sig[os4];
            os4 += zm_next_sig(L, k - 3, plane);
        }
        __builtin_amdgcn_sched_barrier(0);
        in[cur].template load<SIG>(L, o, os, half, half_s);
        advance(k + 2);
        zm_push(idg, tab.at(k, 0));
        zm_push(cx, tab.at(k, 2));
        zm_push(cm, tab.at(k, 3));
        zm_push(cp, tab.at(k, 4));
        zm_push(rr, v.r0);
        zm_push(rb, v.r1);
        const ZmIv<T, SIG> iv{ivp, idg};
        if (SIG) {
            T v0 = idg[0], v1 = idg[0];
            if (has_sig(L, k)) {
                const T dg = tab.at(k, 1);
                v0 = T(1) / (dg + v.s0);
                v1 = T(1) / (dg + v.s1);
            }
            iv.put(0, k, v0);
            iv.put(1, k, v1);
            if (k == c.k0) {
#pragma unroll
                for (int q = 1; q < 4; ++q) {              // planes below the march
                    iv.put(0, k - q, T(0));
                    iv.put(1, k - q, T(0));
                }
            }
        }
        // red, plane k, from a zero start
        zm_push(a0, zm_gs(rr[0], iv.get(L, 0, k, 0)));
        buf(0, cur)[c.lp] = a0[0];
        zm_fence<T, SIG>();
        // black, plane k - 1
        zm_push(b0, zm_gs(rb[1] + zm_nb(buf(0, prv), c, c.x[cur], cx[1], cm[1], cp[1], a0[1], a0[2], a0[0]), iv.get(L, 1, k, 1)));
        buf(1, cur)[c.lp] = b0[0];
        zm_fence<T, SIG>();
        // red, plane k - 2, and black, plane k - 3: a light cycle passes the first sweep's values through
        const T a1n = zm_gs(rr[2] + zm_nb(buf(1, prv), c, c.x[cur], cx[2], cm[2], cp[2], b0[1], b0[2], b0[0]), iv.get(L, 0, k, 2));
        zm_push(a1, two ? a1n : a0[2]);
        buf(2, cur)[c.lp] = a1[0];
        zm_fence<T, SIG>();
        const T b1n = zm_gs(rb[3] + zm_nb(buf(2, prv), c, c.x[cur], cx[3], cm[3], cp[3], a1[1], a1[2], a1[0]), iv.get(L, 1, k, 3));
        zm_push(b1, two ? b1n : b0[2]);
        buf(3, cur)[c.lp] = b1[0];
        zm_fence<T, SIG>();
        // red residual, plane k - 4, and the restriction's sums: the odd row's last
        T d4 = tab.at(k - 4, 1);
        if (SIG) d4 = has_sig(L, k - 4) ? d4 + s4c : d4;
        const T res = res_value(rr[4], d4, a1[2], zm_nb(buf(3, prv), c, c.x[cur], cx[4], cm[4], cp[4], b1[1], b1[2], b1[0]));
        const int p = k - 5;
        const double sp = fmad(wz_of(p), (double)buf(4, prv)[c.lp + kZmP], sr);
        sr = fmad(wz_of(k - 4), (double)res, cur ? sp : 0.0);
        buf(4, cur)[c.lp] = res;
        if (c.own && k - 3 >= c.z0 && k - 3 < c.z1) ealt[(k - 3) * plane + c.q0] = b1[0];
        if ((!cur || p == nz - 1) && own_c && p >= c.z0 && p < c.z1) C.r[cidx(C, gI, gJ, p >> 1)] = (T)(sp * 0.25);
        if (SIG) {
            // sigma of plane k - 1's odd row, then of plane k: the pair's cells in x order
            if (has_sig(L, k - 1)) {
                const double wz = wz_of(k - 1);
                ss = fmad(wz, (double)buf(5, prv)[c.lp + kZmP], ss);
                ss = fmad(wz, (double)buf(6, prv)[c.lp + kZmP], ss);
                if ((!cur || !has_sig(L, k)) && own_c && k - 1 >= c.z0 && k - 1 < c.z1)
                    C.sig[sidx(C, gI, gJ, (k - 1) >> 1)] = (T)(ss * 0.25);
            }
            if (has_sig(L, k)) {
                const bool sw = ((c.row + cur) & 1) != 0;  // the black cell comes first
                const T sa = sw ? v.s1 : v.s0, sb = sw ? v.s0 : v.s1;
                const double wz = wz_of(k);
                ss = fmad(wz, (double)sa, cur && has_sig(L, k - 1) ? ss : 0.0);
                ss = fmad(wz, (double)sb, ss);
                buf(5, cur)[c.lp] = sa;
                buf(6, cur)[c.lp] = sb;
            }
        }
        __syncthreads();
    };
    zm_march(L, c.k0, k1, step);
}

template <typename T, int FINEST>
__global__ __launch_bounds__(kZmThreads) void k_post_zm(const Inst<T> *I, Work w, int level, int nu, int zl) {
    extern __shared__ double tb_raw[];
    const Blk b = find_block(w);
    const Inst<T> &a = I[b.inst];
    const GState *st = wstate(w, b.inst);
    const int done = st->done, light = st->light;
    if (!b.ok | (done != 0) | (level < 0)) return;  // one exit test: see smooth_kernel
    const bool two = nu > 1 && !light;              // the second sweep is made
    const Lv<T, 1> L = zm_view(a.lv[level]), C = gview(a.lv[level + 1]);
    const Xv<T> X = xview(a.xf[level]);
    const ZmBlk c = zm_block(L, b.t, zl);
    const int k1 = c.z1 + kZmH;
    const int nz = L.nz, plane = (L.nx >> 1) * L.ny, half = plane * nz;
    const T FX_AS(1) *ealt = asp<1>(a.lv[level].ealt);
    // LDS: double-buffered planes of the corrected black values and three half-sweeps; a ring of
    // four coarse planes; tables
    T FX_AS(3) *lds = asp<3>((T *)tb_raw);
    auto buf = [&](int stage, int par) { return lds + (2 * stage + par) * kZmA; };
    const int FX_AS(1) *pflags = asp<1>(a.pflags);
    T FX_AS(3) *cbuf = lds + 8 * kZmA;
    T FX_AS(3) *ivp = cbuf + 4 * kZmCW * kZmCW + c.lp - kZmPad;
    const ZmTab<T> tab{cbuf + 4 * kZmCW * kZmCW + 8 * kZmN, c.k0, kZmTab(zl)};
    T FX_AS(3) *wt = tab.p + 5 * kZmTab(zl);               // z weights of the parent and the neighbour plane, clipped planes
    zm_clear(lds, 8 * kZmA);
    tab.fill(L);
    for (int q = threadIdx.x; q < kZmTab(zl); q += kZmThreads) {
        const int k = c.k0 + q;
        wt[3 * q] = k < nz ? X.pwa[k] : T(0);
        wt[3 * q + 1] = k < nz && X.pkb[k] >= 0 ? X.pwb[k] : T(0);
        if (FINEST) wt[3 * q + 2] = k < nz && (pflags[k] & PF_SC) ? T(1) : T(0);
    }
    // coarse planes: one value per thread
    const int cq = min((int)threadIdx.x, kZmCW * kZmCW - 1), cj = cq / kZmCW, ci = cq - cj * kZmCW;
    int CI = c.tx * (kZmT / 2) - kZmH / 2 - 1 + ci, CJ = c.ty * (kZmT / 2) - kZmH / 2 - 1 + cj;
    CI = (CI % C.nx + C.nx) % C.nx;
    CJ = (CJ % C.ny + C.ny) % C.ny;
    auto cload = [&](int K) { return C.e[cidx(C, CI, CJ, max(0, min(K, C.nz - 1)))]; };
    auto cstore = [&](int K, T v) {
        if (threadIdx.x < kZmCW * kZmCW) cbuf[(K & 3) * (kZmCW * kZmCW) + threadIdx.x] = v;
    };
    const int K0 = c.k0 >> 1;
    {
        const T v0 = cload(K0 - 1), v1 = cload(K0), v2 = cload(K0 + 1);
        cstore(K0 - 1, v0);
        cstore(K0, v1);
        cstore(K0 + 1, v2);
    }
    T cnext = cload(K0 + 2);
    // the thread's coarse operands: its column, the x neighbour on either side, the y neighbour's row
    const int co = (1 + (c.row >> 1)) * kZmCW + 1 + c.m, cy = (c.row & 1) ? kZmCW : -kZmCW;
    const T wx[2] = {T(0.75), T(0.25)}, wy[2] = {T(0.75), T(0.25)};
    T wgt[2][2];
#pragma unroll
    for (int yy = 0; yy < 2; ++yy)
#pragma unroll
        for (int xx = 0; xx < 2; ++xx) wgt[yy][xx] = wx[xx] * wy[yy];
    auto lateral = [&](int K, int dx) {
        const T FX_AS(3) *p = cbuf + (K & 3) * (kZmCW * kZmCW) + co;
        T v[2][2];
        v[0][0] = p[0];
        v[0][1] = p[dx];
        v[1][0] = p[cy];
        v[1][1] = p[cy + dx];
        return lint_xy<2, 2>(wgt, v);
    };
    T rr[4] = {}, rb[5] = {}, e0[3] = {}, a0[3] = {}, b0[3] = {}, a1[3] = {};
    T cx[5] = {}, cm[5] = {}, cp[5] = {}, idg[5] = {};
    ZmIn<T> in[2];
    T eb[2];
    // cell indices of the planes loaded next: k + 2 of a step
    const int half_s = plane * (L.sig_hi - L.sig_lo);
    int o = c.k0 * plane + c.q0, os = zm_first_sig(L, c.k0, plane) + c.q0;
    auto advance = [&](int k) {
        o += zm_next(L, k, plane);
        os += zm_next_sig(L, k, plane);
    };
    const bool any_sig = zm_sig(L, c.k0, k1);
    for (int q = 0; q < 2; ++q) {
        if (any_sig) in[q].template load<1>(L, o, os, half, half_s);
        else in[q].template load<0>(L, o, os, half, half_s);
        eb[q] = ealt[o];
        advance(c.k0 + q);
    }
    const size_t off = (size_t)a.kb * a.nx * a.ny;
    const double FX_AS(1) *phi_in = nullptr;
    double FX_AS(1) *phi_out = nullptr;
    const size_t nxy = (size_t)L.nx * L.ny;
    const double dmax = a.dmax;
    dpair ph = {};                                         // phi of the plane that is finished next
    if (FINEST) {
        phi_in = asp<1>(a.phi[cyc_src(st)]) + off + max(c.k0 - 3, 0) * nxy + 2 * c.q0;
        phi_out = asp<1>(a.phi[cyc_dst(st)]) + off + 2 * c.q0;
    }
    // the loads above are waited for here: the march's own waits then count its own loads
    __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0)
    __syncthreads();                                       // tables, coarse planes
    auto step = [&](int k, int cur, auto sig_) {
        constexpr int SIG = decltype(sig_)::value;
        const int prv = cur ^ 1;                           // k0 is even: cur is the plane's parity
        // waits are in the order of issue: what is needed soonest is loaded first
        const dpair phk = zm_take(ph);
        const ZmIn<T> v = in[cur].template take<SIG>();
        const T ebk = zm_take(eb[cur]);
        if (FINEST) {
            ph = *(const dpair FX_AS(1) *)phi_in;
            phi_in += k >= 3 && k - 2 < nz ? nxy : 0;      // the plane finished in the step after the next
        }
        __builtin_amdgcn_sched_barrier(0);
        in[cur].template load<SIG>(L, o, os, half, half_s);
        eb[cur] = ealt[o];
        advance(k + 2);
        zm_push(idg, tab.at(k, 0));
        zm_push(cx, tab.at(k, 2));
        zm_push(cm, tab.at(k, 3));
        zm_push(cp, tab.at(k, 4));
        zm_push(rr, v.r0);
        zm_push(rb, v.r1);
        const ZmIv<T, SIG> iv{ivp, idg};
        const T iv4 = iv.get(L, 1, k, 4);                  // ahead of its slot's next value
        if (SIG) {
            T v0 = idg[0], v1 = idg[0];
            if (has_sig(L, k)) {
                const T dg = tab.at(k, 1);
                v0 = T(1) / (dg + v.s0);
                v1 = T(1) / (dg + v.s1);
            }
            iv.put(0, k, v0);
            iv.put(1, k, v1);
            if (k == c.k0) {
#pragma unroll
                for (int q = 1; q < 4; ++q) {              // planes below the march
                    iv.put(0, k - q, T(0));
                    iv.put(1, k - q, T(0));
                }
            }
        }
        // corrected black value, plane k: the black cell is at 2m + (1 + row + k) % 2
        {
            const int K = k >> 1, Kn = cur ? K + 1 : K - 1;
            const int dx = ((c.row + cur) & 1) ? -1 : 1;
            const T wa = uniform_value((T)wt[3 * (k - c.k0)]), wb = uniform_value((T)wt[3 * (k - c.k0) + 1]);
            zm_push(e0, ebk + lint_z(wa, lateral(K, dx), wb, lateral(Kn, dx)));
        }
        buf(0, cur)[c.lp] = e0[0];
        zm_fence<T, SIG>();
        // red, plane k - 1
        zm_push(a0, zm_gs(rr[1] + zm_nb(buf(0, prv), c, c.x[prv], cx[1], cm[1], cp[1], e0[1], e0[2], e0[0]), iv.get(L, 0, k, 1)));
        buf(1, cur)[c.lp] = a0[0];
        zm_fence<T, SIG>();
        // black, plane k - 2
        zm_push(b0, zm_gs(rb[2] + zm_nb(buf(1, prv), c, c.x[prv], cx[2], cm[2], cp[2], a0[1], a0[2], a0[0]), iv.get(L, 1, k, 2)));
        buf(2, cur)[c.lp] = b0[0];
        zm_fence<T, SIG>();
        // red, plane k - 3, and black, plane k - 4 (light: passed through)
        const T a1n = zm_gs(rr[3] + zm_nb(buf(2, prv), c, c.x[prv], cx[3], cm[3], cp[3], b0[1], b0[2], b0[0]), iv.get(L, 0, k, 3));
        zm_push(a1, two ? a1n : a0[2]);
        buf(3, cur)[c.lp] = a1[0];
        zm_fence<T, SIG>();
        const T b1n = zm_gs(rb[4] + zm_nb(buf(3, prv), c, c.x[prv], cx[4], cm[4], cp[4], a1[1], a1[2], a1[0]), iv4);
        const T fb = two ? b1n : b0[2];
        // the finished pair, plane k - 4
        const T fr = a1[1];
        const int p = k - 4;
        if (c.own && p >= c.z0 && p < c.z1) {
            if (FINEST) {
                const double lim = uniform_value((T)wt[3 * (p - c.k0) + 2]) != T(0) ? dmax : 1e300;
                const double db = fmin(fmax((double)fb, -lim), lim), dr = fmin(fmax((double)fr, -lim), lim);
                const bool odd = ((c.row + cur) & 1) == 0;         // the black cell is the pair's second
                dpair v2;
                v2.x = phk.x + (odd ? dr : db);
                v2.y = phk.y + (odd ? db : dr);
                *(dpair FX_AS(1) *)(phi_out + p * nxy) = v2;
            } else {
                L.e[p * plane + c.q0] = fr;
                L.e[half + p * plane + c.q0] = fb;
            }
        }
        // coarse plane K + 2 joins the ring for the next pair of planes
        if (cur) {
            cstore((k >> 1) + 2, zm_take(cnext));
            cnext = cload((k >> 1) + 3);
        }
        __syncthreads();
    };
    zm_march(L, c.k0, k1, step);
}

// --------------------------------------------- coarse levels in one workgroup
// Quotient q / d for 0 <= q < 2^20 and 1 <= d without an integer division: (q + 1/2) / d
// lies at least 1/(2d) from the next integer, while the rounded product is off by at most
// 2^-22 q/d (every level of the coarse kernel has fewer than 2^14 cells).
struct FDiv {
    int d;
    float inv;
};
__device__ __forceinline__ FDiv fdiv_of(int d) { return {d, 1.0f / (float)d}; }
__device__ __forceinline__ int fquo(int q, const FDiv &f) { return (int)(((float)q + 0.5f) * f.inv); }

// (i, j, k) of natural index c on an nx x ny x nz level
struct Split3 {
    FDiv fx, fy;
};
__device__ __forceinline__ void split_c(int c, const Split3 &s, int &i, int &j, int &k) {
    const int row = fquo(c, s.fx);
    i = c - row * s.fx.d;
    k = fquo(row, s.fy);
    j = row - k * s.fy.d;
}

constexpr int kCoarseThreads = 1024;
// First thread of this wave.  Waves without cells on a level skip its phases (but not the
// barriers): the arithmetic of fifteen idle waves would hold up the one that has some.
__device__ __forceinline__ int wave_first() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x & ~63); }

// The workers of a level: the whole workgroup, or (W = 1) its first wave alone, where a level and
// everything below it fit a wave; its LDS accesses complete in order, so a phase needs no
// barrier there.
template <int W>
struct Crew {
    static constexpr int size = W ? 64 : kCoarseThreads;
    static __device__ __forceinline__ void sync() {
        if (W) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    }
};

// 1 / x for a positive normal x, to within a rounding or two of the quotient (hardware
// estimate and Newton steps).  A division is about 400 cycles of latency, this 100; the coarse
// levels need no kernel's bits but their own.
__device__ __forceinline__ double rcp_newton(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
    return __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
}
__device__ __forceinline__ float rcp_newton(float x) { return 1.0f / x; }

// A coarse-kernel phase: the crew works on the level's cells, and a barrier separates it from
// the next phase.  A phase is latency: one chain of LDS reads, FP64 arithmetic and a store, so
// what a thread needs of its cells for all sweeps of a level (right-hand sides, reciprocal
// diagonals, coefficients, neighbour offsets) is worked out once and held in registers.
//
// Red/black level: NP storage pairs (a red and a black cell of one row) per thread.  The
// pair's red and black cells are each other's x neighbours; their other x neighbour lies in
// the pair dx away, the y and z neighbours in pairs oy, oz away (all in the other colour's
// array).  Absent neighbours (z-ends, ny = 1) weigh 0 and point at the pair itself.
template <typename T, int NP, int W>
struct RbCells {
    T r[2][NP], iv[2][NP], cx[NP], cy[NP], cm[NP], cp[NP], d0[NP];
    int q[NP], dx[2][NP], oy[2][NP], oz[2][NP];
    bool on[NP];
    bool act;                                          // this wave has cells

    __device__ __forceinline__ void load(const Lv<T, 3> &L) {
        const int hx = L.nx >> 1, plane = hx * L.ny, n = plane * L.nz;
        const int hsz = plane * (L.sig_hi - L.sig_lo);
        act = W || wave_first() < n;
        if (!act) return;
        const Split3 sp{fdiv_of(hx), fdiv_of(L.ny)};
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int c = threadIdx.x + p * Crew<W>::size;
            on[p] = c < n;
            q[p] = on[p] ? c : 0;
            int m, j, k;
            split_c(q[p], sp, m, j, k);
            const int par = (j + k) & 1;               // the red cell is at 2m + par
            const int up = m + 1 == hx ? 1 - hx : 1, dn = m == 0 ? hx - 1 : -1;
            dx[0][p] = par ? up : dn;
            dx[1][p] = par ? dn : up;
            oy[0][p] = L.ny > 1 ? (wrap_p(j, L.ny) - j) * hx : 0;
            oy[1][p] = L.ny > 1 ? (wrap_m(j, L.ny) - j) * hx : 0;
            oz[0][p] = k > 0 ? -plane : 0;
            oz[1][p] = k < L.nz - 1 ? plane : 0;
            cx[p] = L.cxy[k];
            cy[p] = L.ny > 1 ? cx[p] : T(0);
            cm[p] = k > 0 ? L.czm[k] : T(0);
            cp[p] = k < L.nz - 1 ? L.czp[k] : T(0);
            const bool hs = k >= L.sig_lo && k < L.sig_hi;
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) {
                r[c2][p] = L.r[c2 * n + q[p]];
                T d = L.dg[k];
                if (hs) d += L.sig[c2 * hsz + q[p] - L.sig_lo * plane];
                if (c2 == 0) d0[p] = d;
                iv[c2][p] = rcp_newton(d);
            }
        }
    }
    // neighbour sum of colour c2's cell of pair p
    __device__ __forceinline__ T nb(const T FX_AS(3) *eo, int c2, int p) const {
        const T FX_AS(3) *e = eo + q[p];
        return nb6(cx[p], cy[p], cm[p], cp[p], e[0], e[dx[c2][p]], e[oy[0][p]], e[oy[1][p]], e[oz[0][p]], e[oz[1][p]]);
    }
    __device__ __forceinline__ void half_sweep(const Lv<T, 3> &L, int c2, int zero_init) const {
        const int n = (L.nx >> 1) * L.ny * L.nz;
        T FX_AS(3) *es = L.e + c2 * n;
        const T FX_AS(3) *eo = L.e + (1 - c2) * n;
        if (act) {
            T v[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) v[p] = (zero_init ? r[c2][p] : r[c2][p] + nb(eo, c2, p)) * iv[c2][p];
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (on[p]) es[q[p]] = v[p];
        }
        Crew<W>::sync();
    }
    // the red cells' residual into their own e (dead until the next red half-sweep)
    __device__ __forceinline__ void red_residual(const Lv<T, 3> &L) const {
        const int n = (L.nx >> 1) * L.ny * L.nz;
        if (act) {
            T v[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) v[p] = res_value(r[0][p], d0[p], L.e[q[p]], nb(L.e + n, 0, p));
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (on[p]) L.e[q[p]] = v[p];
        }
        Crew<W>::sync();
    }
};

// Restriction of a red/black level halved in x and y from the red residuals just formed: the
// red child of row (j, k) of coarse column I is the red cell of pair I of that row.
template <int W, typename T, typename X_>
__device__ __forceinline__ void restrict_pairs(const Lv<T, 3> &F, const Lv<T, 3> &C, const X_ &X) {
    const int hx = F.nx >> 1, n = C.nx * C.ny * C.nz;
    const Split3 sp{fdiv_of(C.nx), fdiv_of(C.ny)};
    for (int c = threadIdx.x; c < n; c += Crew<W>::size) {
        int I, J, K;
        split_c(c, sp, I, J, K);
        const int ks = X.cks[K], cnt = X.ccnt[K];
        const double it = rcp_newton((double)X.cthick[K]);
        double sr = 0.0, ss = 0.0;
        for (int dz = 0; dz < cnt; ++dz) {
            const int k = ks + dz;
            const double wz = (double)X.fthick[k] * it;
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
                const int j = 2 * J + dy;
                sr += wz * (double)F.e[(k * F.ny + j) * hx + I];
                if (has_sig(F, k)) {
#pragma unroll
                    for (int dx = 0; dx < 2; ++dx) ss += wz * (double)F.sig[sidx(F, 2 * I + dx, j, k)];
                }
            }
        }
        C.r[cidx(C, I, J, K)] = (T)(sr * 0.25);
        if (has_sig(C, K)) C.sig[sidx(C, I, J, K)] = (T)(ss * 0.25);
    }
    Crew<W>::sync();
}

template <typename T, int NP, int W, typename X_>
__device__ __forceinline__ void co_pre_rb(const Lv<T, 3> &L, const Lv<T, 3> &C, const X_ &X, int nu) {
    RbCells<T, NP, W> c;
    c.load(L);
    for (int s = 0; s < nu; ++s) {
        c.half_sweep(L, 0, s == 0);
        c.half_sweep(L, 1, 0);
    }
    if (X.xy == 1) {
        c.red_residual(L);
        restrict_pairs<W>(L, C, X);
    }
}
template <typename T, int NP, int W>
__device__ __forceinline__ void co_post_rb(const Lv<T, 3> &L, int nu) {
    RbCells<T, NP, W> c;
    c.load(L);
    for (int s = 0; s < nu; ++s) {
        c.half_sweep(L, 0, 0);
        c.half_sweep(L, 1, 0);
    }
}

// Plainly stored level: NP cells per thread, each of one of the four colours.  With x and y both
// odd the corner cell of a plane shares its colour with two of its periodic neighbours: a
// barrier between the values and their stores then keeps the sweep reproducible.
template <typename T, int NP, int W>
struct NatCells {
    T r[NP], iv[NP], cx[NP], cm[NP], cp[NP];
    int c[NP], ox[2][NP], oy[2][NP], oz[2][NP], col[NP];   // col -1: no cell
    bool act;                                              // this wave has cells

    __device__ __forceinline__ void load(const Lv<T, 3> &L) {
        const int plane = L.nx * L.ny, n = plane * L.nz;
        act = W || wave_first() < n;
        if (!act) return;
        const Split3 sp{fdiv_of(L.nx), fdiv_of(L.ny)};
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int cc = threadIdx.x + p * Crew<W>::size;
            const bool on = cc < n;
            c[p] = on ? cc : 0;
            int i, j, k;
            split_c(c[p], sp, i, j, k);
            ox[0][p] = wrap_p(i, L.nx) - i;
            ox[1][p] = wrap_m(i, L.nx) - i;
            oy[0][p] = (wrap_p(j, L.ny) - j) * L.nx;
            oy[1][p] = (wrap_m(j, L.ny) - j) * L.nx;
            oz[0][p] = k > 0 ? -plane : 0;
            oz[1][p] = k < L.nz - 1 ? plane : 0;
            col[p] = on ? nat_color(L, i, j, k) : -1;
            cx[p] = L.cxy[k];
            cm[p] = k > 0 ? L.czm[k] : T(0);
            cp[p] = k < L.nz - 1 ? L.czp[k] : T(0);
            r[p] = L.r[c[p]];
            iv[p] = rcp_newton(diag_of(L, i, j, k));
        }
    }
    __device__ __forceinline__ void sweep(const Lv<T, 3> &L, int zero_init) const {
        const T wx = L.nx > 1 ? T(1) : T(0), wy = L.ny > 1 ? T(1) : T(0);
        const bool corner = (L.nx & L.ny & 1) != 0;
        for (int color = 0; color < 4; ++color) {
            const int zi = zero_init && color == 0;
            T v[NP];
            if (act) {
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    v[p] = T(0);
                    if (col[p] != color) continue;
                    T s = 0;
                    if (!zi) {
                        const T FX_AS(3) *e = L.e + c[p];
                        const T x = wx * (e[ox[0][p]] + e[ox[1][p]]), y = wy * (e[oy[0][p]] + e[oy[1][p]]);
                        s = fmad(cp[p], e[oz[1][p]], fmad(cm[p], e[oz[0][p]], fmad(cx[p], y, cx[p] * x)));
                    }
                    v[p] = (r[p] + s) * iv[p];
                }
            }
            if (corner) Crew<W>::sync();
            if (act) {
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    if (col[p] == color || (zi && col[p] >= 0)) L.e[c[p]] = v[p];
            }
            Crew<W>::sync();
        }
    }
};
template <typename T, int NP, int W>
__device__ __forceinline__ void co_smooth_nat(const Lv<T, 3> &L, int nu, int zero_init) {
    NatCells<T, NP, W> c;
    c.load(L);
    for (int s = 0; s < nu; ++s) c.sweep(L, zero_init && s == 0);
}

// Pre-smoothing and restriction, and prolongation and post-smoothing, of one level.  A red/black
// level here holds e and r in kCoarseLdsBytes, so at most 4096 cells in FP64 and 8192 in FP32.  A
// plainly stored one is halved in z alone: with the levels below it (half of it, a quarter, ..., the
// bottom's four vectors) it takes four vectors of its cells, so at most 4096 where all fit
// kCoarseLdsBytes, and kCoarseNatCells where they take more.
static_assert(kCoarseLdsBytes / (2 * sizeof(double)) <= 4 * kCoarseThreads &&
                  kCoarseLdsBytes / (2 * sizeof(float)) <= 8 * kCoarseThreads &&
                  kCoarseLdsBytes / (4 * sizeof(float)) <= 4 * kCoarseThreads && kCoarseNatCells <= 4 * kCoarseThreads,
              "cells per thread");
template <typename T>
__device__ __forceinline__ void co_nat(const Lv<T, 3> &L, int nu, int zero_init) {
    const int n = L.nx * L.ny * L.nz;
    if (n <= kCoarseThreads) co_smooth_nat<T, 1, 0>(L, nu, zero_init);
    else if (n <= 2 * kCoarseThreads) co_smooth_nat<T, 2, 0>(L, nu, zero_init);
    else co_smooth_nat<T, 4, 0>(L, nu, zero_init);
}
template <int W, typename T, typename X_>
__device__ __forceinline__ void co_down(const Lv<T, 3> &L, const Lv<T, 3> &C, const X_ &X, int nu) {
    if (L.rb) {
        const int n = (L.nx >> 1) * L.ny * L.nz;
        if (W || n <= kCoarseThreads) co_pre_rb<T, 1, W>(L, C, X, nu);
        else if (n <= 2 * kCoarseThreads) co_pre_rb<T, 2, W>(L, C, X, nu);
        else if constexpr (sizeof(T) == 4 && !W) co_pre_rb<T, 4, W>(L, C, X, nu);
        if (X.xy == 1) return;
    } else if (W) {
        co_smooth_nat<T, 1, W>(L, nu, 1);
    } else {
        co_nat(L, nu, 1);
    }
    const int n = C.nx * C.ny * C.nz;
    const Split3 sp{fdiv_of(C.nx), fdiv_of(C.ny)};
    for (int c = threadIdx.x; c < n; c += Crew<W>::size) {
        int I0, J0, K0;
        split_c(c, sp, I0, J0, K0);
        restrict_cell(L, C, X, I0, J0, K0);
    }
    Crew<W>::sync();
}
template <int W, typename T, typename X_>
__device__ __forceinline__ void co_up(const Lv<T, 3> &L, const Lv<T, 3> &C, const X_ &X, int nu) {
    if (L.rb) {
        const int hx = L.nx >> 1;
        const int n = hx * L.ny * L.nz;
        T FX_AS(3) *eb = L.e + n;
        const Split3 sp{fdiv_of(hx), fdiv_of(L.ny)};
        for (int q = threadIdx.x; q < n; q += Crew<W>::size) {
            int m, j, k;
            split_c(q, sp, m, j, k);
            const int i = 2 * m + ((1 + j + k) & 1);
            const T v = X.xy == 1 ? prolong_value<1>(C, X, i, j, k)
                        : X.xy == 2 ? prolong_value<2>(C, X, i, j, k) : prolong_value<0>(C, X, i, j, k);
            eb[q] += v;
        }
        Crew<W>::sync();
        if (W || n <= kCoarseThreads) co_post_rb<T, 1, W>(L, nu);
        else if (n <= 2 * kCoarseThreads) co_post_rb<T, 2, W>(L, nu);
        else if constexpr (sizeof(T) == 4 && !W) co_post_rb<T, 4, W>(L, nu);
    } else {
        const int n = L.nx * L.ny * L.nz;
        const Split3 sp{fdiv_of(L.nx), fdiv_of(L.ny)};
        for (int c = threadIdx.x; c < n; c += Crew<W>::size) {
            int i, j, k;
            split_c(c, sp, i, j, k);
            prolong_cell(L, C, X, i, j, k);
        }
        Crew<W>::sync();
        if (W) co_smooth_nat<T, 1, W>(L, nu, 0);
        else co_nat(L, nu, 0);
    }
}

// Sum over the 64 lanes of a wave in a fixed order with DPP adds (row shifts, then the two
// row broadcasts leave the total in lane 63); every lane gets the same bits.  Six shuffles
// through the LDS unit took several times as long.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0x111, 0xf>(v);                        // row_shr 1, 2, 4, 8
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);                        // row_bcast 15, 31
    v = dpp_add<0x143, 0xc>(v);
    return lane_value(v, 63);
}

// Two sums over the workgroup in a fixed order; every thread gets the totals.  red holds a pair of
// partials per wave (act: this wave has terms); the caller's next write to it comes after
// another barrier.
__device__ __forceinline__ void block_totals(double &x, double &y, double FX_AS(3) *red, bool act) {
    constexpr int NW = kCoarseThreads / 64;
    static_assert(NW == 16, "a partial per lane of a row of 16");
    if (act) {
        x = wave_sum(x);
        y = wave_sum(y);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        red[wave] = act ? x : 0.0;
        red[NW + wave] = act ? y : 0.0;
    }
    __syncthreads();
    double v = red[lane & (2 * NW - 1)];                   // row 0 the x partials, row 1 those of y
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    x = lane_value(v, 15);
    y = lane_value(v, 31);
}

// Bottom solve on the coarsest level: conjugate gradients on the symmetric
// positive definite (L + diag sigma) e = r from e = 0, until the residual has
// dropped by sqrt(tol2) or after iters steps.  r is overwritten by the
// residual.  Unlike a fixed number of Gauss-Seidel sweeps this also solves
// coarsest levels that keep many cells in x and y (odd lateral sizes stop the
// x-y coarsening early).
// The same conjugate gradients for a bottom level of at most 64 cells, run by
// the first wave alone with one cell per lane: the operator's neighbours are
// read from other lanes' registers, the dot products are wave sums, and no
// workgroup barrier is needed inside the iteration.
template <typename T>
__device__ void bottom_cg_wave(const Lv<T, 3> &B, int iters, double tol2) {
    const int n = B.nx * B.ny * B.nz;
    const int c = threadIdx.x;
    const bool on = c < n;
    int i = 0, j = 0, k = 0;
    if (on) {
        const Split3 sp{fdiv_of(B.nx), fdiv_of(B.ny)};
        split_c(c, sp, i, j, k);
    }
    // neighbour lanes (natural order) and coefficients; absent neighbours weigh 0
    int nl[6];
    double w[6];
    const double cx = on ? (double)B.cxy[k] : 0.0;
    nl[0] = (k * B.ny + j) * B.nx + wrap_p(i, B.nx);
    nl[1] = (k * B.ny + j) * B.nx + wrap_m(i, B.nx);
    w[0] = w[1] = B.nx > 1 ? cx : 0.0;
    nl[2] = (k * B.ny + wrap_p(j, B.ny)) * B.nx + i;
    nl[3] = (k * B.ny + wrap_m(j, B.ny)) * B.nx + i;
    w[2] = w[3] = B.ny > 1 ? cx : 0.0;
    nl[4] = k > 0 ? c - B.nx * B.ny : c;
    w[4] = on && k > 0 ? (double)B.czm[k] : 0.0;
    nl[5] = k < B.nz - 1 ? c + B.nx * B.ny : c;
    w[5] = on && k < B.nz - 1 ? (double)B.czp[k] : 0.0;
    const int ci = on ? cidx(B, i, j, k) : 0;
    const double d = on ? (double)diag_of(B, i, j, k) : 1.0;
    double r = on ? (double)B.r[ci] : 0.0;
    double x = 0.0, p = r;
    double rr = wave_sum(r * r);
    const double stop = tol2 * rr;
    for (int it = 0; it < iters && rr > stop; ++it) {
        double q = d * p;
#pragma unroll
        for (int m = 0; m < 6; ++m) q -= w[m] * __shfl(p, nl[m], 64);
        if (!on) q = 0.0;
        const double pq = wave_sum(p * q);
        if (!(pq > 0.0)) break;
        const double alpha = rr / pq;
        x += alpha * p;
        r -= alpha * q;
        const double rn = wave_sum(r * r);
        const double beta = rn / rr;
        rr = rn;
        p = r + beta * p;
    }
    if (on) {
        B.e[ci] = (T)x;
        B.r[ci] = (T)r;
    }
}

// A bottom level of at most 8 cells, solved directly by the first wave: lane 8 i + j holds the
// matrix entry (i, j), every lane of row i the right-hand side; Gauss-Jordan without pivoting
// (the matrix is symmetric positive definite), a step per cell.  Bound by the latency of its
// steps, about 300 cycles each; the conjugate gradients took 2500 a step (22000 cycles of the
// 16 x 16 x 20 stack's 63000 on its 8 cells).
template <typename T>
__device__ __forceinline__ void bottom_direct(const Lv<T, 3> &B) {
    const int n = B.nx * B.ny * B.nz, plane = B.nx * B.ny;
    const int lane = threadIdx.x, row = lane >> 3, col = lane & 7;
    const bool on = row < n;
    const int c = on ? row : 0;
    const Split3 sp{fdiv_of(B.nx), fdiv_of(B.ny)};
    int i, j, k;
    split_c(c, sp, i, j, k);
    const double cx = (double)B.cxy[k];
    const double wx = B.nx > 1 ? cx : 0.0, wy = B.ny > 1 ? cx : 0.0;
    const int base = c - i;
    double a = 0.0;
    a -= base + wrap_p(i, B.nx) == col ? wx : 0.0;
    a -= base + wrap_m(i, B.nx) == col ? wx : 0.0;
    a -= k * plane + wrap_p(j, B.ny) * B.nx + i == col ? wy : 0.0;
    a -= k * plane + wrap_m(j, B.ny) * B.nx + i == col ? wy : 0.0;
    a -= k > 0 && c - plane == col ? (double)B.czm[k] : 0.0;
    a -= k < B.nz - 1 && c + plane == col ? (double)B.czp[k] : 0.0;
    if (c == col) a += (double)diag_of(B, i, j, k);
    if (!on) a = row == col ? 1.0 : 0.0;
    const int ci = cidx(B, i, j, k);
    double x = on ? (double)B.r[ci] : 0.0;
    for (int p = 0; p < n; ++p) {
        const double inv = rcp_newton(__shfl(a, 9 * p, 64));
        const double ar = __shfl(a, 8 * p + col, 64) * inv, xr = __shfl(x, 8 * p, 64) * inv;
        const double f = __shfl(a, 8 * row + p, 64);
        a = row == p ? ar : __builtin_fma(-f, ar, a);
        x = row == p ? xr : __builtin_fma(-f, xr, x);
    }
    if (on && col == 0) B.e[ci] = (T)x;
}

// A thread per cell, NP cells each; the vectors stay in registers, the residual is shared through
// LDS (rs).  The recurrences are Chronopoulos and Gear's (1989): with w = A r, both inner
// products of a step, (r, r) and (w, r), are summed together, so a step is one exchange of r
// and one reduction, two barriers (about 1000 cycles; three exchanges and sums of 16 partials
// in sequence took 2200).
template <typename T, int NP>
__device__ __forceinline__ void bottom_cg_block(const Lv<T, 3> &B, T FX_AS(3) *rs, double FX_AS(3) *red, int iters,
                                                double tol2) {
    const int n = B.nx * B.ny * B.nz, plane = B.nx * B.ny;
    const Split3 sp{fdiv_of(B.nx), fdiv_of(B.ny)};
    double r[NP], x[NP], d[NP], p[NP], s[NP], cx[NP], cy[NP], cm[NP], cp[NP];
    int c[NP], ci[NP], ox[2][NP], oy[2][NP], oz[2][NP];
    bool on[NP];
    const bool act = wave_first() < n;
    if (act) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int cc = threadIdx.x + u * kCoarseThreads;
            on[u] = cc < n;
            c[u] = on[u] ? cc : 0;
            int i, j, k;
            split_c(c[u], sp, i, j, k);
            ci[u] = cidx(B, i, j, k);
            ox[0][u] = wrap_p(i, B.nx) - i;
            ox[1][u] = wrap_m(i, B.nx) - i;
            oy[0][u] = (wrap_p(j, B.ny) - j) * B.nx;
            oy[1][u] = (wrap_m(j, B.ny) - j) * B.nx;
            oz[0][u] = k > 0 ? -plane : 0;
            oz[1][u] = k < B.nz - 1 ? plane : 0;
            cx[u] = on[u] && B.nx > 1 ? (double)B.cxy[k] : 0.0;
            cy[u] = on[u] && B.ny > 1 ? (double)B.cxy[k] : 0.0;
            cm[u] = on[u] && k > 0 ? (double)B.czm[k] : 0.0;
            cp[u] = on[u] && k < B.nz - 1 ? (double)B.czp[k] : 0.0;
            d[u] = on[u] ? (double)diag_of(B, i, j, k) : 0.0;
            r[u] = on[u] ? (double)B.r[ci[u]] : 0.0;
            x[u] = p[u] = s[u] = 0.0;
        }
    }
    double g_old = 1.0, a_old = 1.0, stop = 0.0;
    for (int it = 0; it <= iters; ++it) {
        if (act) {
#pragma unroll
            for (int u = 0; u < NP; ++u)
                if (on[u]) rs[c[u]] = (T)r[u];
        }
        __syncthreads();
        double w[NP], g = 0.0, h = 0.0;
        if (act) {
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const T FX_AS(3) *e = rs + c[u];
                if (on[u]) r[u] = (double)e[0];            // the residual as its neighbours see it
                w[u] = d[u] * r[u] - cx[u] * ((double)e[ox[0][u]] + (double)e[ox[1][u]]) -
                       cy[u] * ((double)e[oy[0][u]] + (double)e[oy[1][u]]) - cm[u] * (double)e[oz[0][u]] -
                       cp[u] * (double)e[oz[1][u]];
                g += r[u] * r[u];
                h += w[u] * r[u];
            }
        }
        block_totals(g, h, red, act);
        if (it == 0) stop = tol2 * g;
        if (!(g > stop) || it == iters) break;
        const double beta = it ? g * rcp_newton(g_old) : 0.0;
        const double den = it ? h - beta * g * rcp_newton(a_old) : h;
        if (!(den > 0.0)) break;
        const double alpha = g * rcp_newton(den);
        g_old = g;
        a_old = alpha;
        if (act) {
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                p[u] = r[u] + beta * p[u];
                s[u] = w[u] + beta * s[u];
                x[u] += alpha * p[u];
                r[u] -= alpha * s[u];
            }
        }
    }
    if (act) {
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (on[u]) B.e[ci[u]] = (T)x[u];
    }
    __syncthreads();
}

// The bottom solve by the whole workgroup (n > 64) or by its first wave.  The coarsest level
// holds e, r and two vectors in kCoarseLdsBytes: at most 2048 cells in FP64 and 4096 in FP32,
// which every instantiation's cells per thread must cover.
static_assert(kCoarseLdsBytes / (4 * sizeof(double)) <= 2 * kCoarseThreads &&
                  kCoarseLdsBytes / (4 * sizeof(float)) <= 4 * kCoarseThreads,
              "cells per thread of the bottom solve");
template <typename T>
__device__ __forceinline__ void bottom_block(const Lv<T, 3> &B, T FX_AS(3) *rs, double FX_AS(3) *red, int iters,
                                             double tol2) {
    const int n = B.nx * B.ny * B.nz;
    if (n <= kCoarseThreads) bottom_cg_block<T, 1>(B, rs, red, iters, tol2);
    else if (n <= 2 * kCoarseThreads) bottom_cg_block<T, 2>(B, rs, red, iters, tol2);
    else if constexpr (sizeof(T) == 4) bottom_cg_block<T, 4>(B, rs, red, iters, tol2);
}
template <typename T>
__device__ __forceinline__ void bottom_wave(const Lv<T, 3> &B, int iters, double tol2) {
    if (B.nx * B.ny * B.nz <= 8) bottom_direct(B);
    else bottom_cg_wave(B, iters, tol2);
}

// A block per instance: the V-cycle from level lc down to the coarsest with
// every level's e, r, sigma and coefficient tables resident in LDS.
template <typename T>
__global__ __launch_bounds__(kCoarseThreads) void k_coarse(const Inst<T> *I, InstState *S) {
    extern __shared__ double lds_raw[];
    const Inst<T> &A = I[blockIdx.x];
    const GState *sta = asp<1>(S + blockIdx.x);
    // read together, one exit test: see smooth_kernel
    const int done = sta->done, light = sta->light, l0 = A.lc, nl = A.nlev - A.lc, qw = A.wave_lev;
    const int nu1 = light ? 1 : A.nu1, nu2 = light ? 1 : A.nu2;
    if ((done != 0) | (l0 < 0)) return;
    unsigned char FX_AS(3) *lds = asp<3>((unsigned char *)lds_raw);
    auto lvl = [&](int q) {
        const LevelArgs<T> &G = A.lv[l0 + q];
        Lv<T, 3> L;
        L.nx = G.nx; L.ny = G.ny; L.nz = G.nz; L.rb = G.rb;
        L.sig_lo = G.sig_lo; L.sig_hi = G.sig_hi;
        L.e = (T FX_AS(3) *)(lds + A.off_e[q]);
        L.r = (T FX_AS(3) *)(lds + A.off_r[q]);
        L.sig = (T FX_AS(3) *)(lds + A.off_s[q]);
        T FX_AS(3) *tab = (T FX_AS(3) *)(lds + A.off_t[q]);
        L.cxy = tab;
        L.czm = tab + L.nz;
        L.czp = tab + 2 * L.nz;
        L.dg = tab + 3 * L.nz;
        return L;
    };
    // transfer tables between levels q and q + 1 in LDS
    auto xlds = [&](int q) {
        const int nf = A.lv[l0 + q].nz, nc = A.lv[l0 + q + 1].nz;
        int FX_AS(3) *ib = (int FX_AS(3) *)(lds + A.off_x[q]);
        Xv<T, 3> X;
        X.cks = ib;
        X.ccnt = ib + nc;
        X.cthick = ib + 2 * nc;
        X.fthick = ib + 3 * nc;
        X.pka = ib + 3 * nc + nf;
        X.pkb = ib + 3 * nc + 2 * nf;
        const T FX_AS(3) *wb =
            (const T FX_AS(3) *)(lds + ((A.off_x[q] + (3 * nc + 3 * nf) * (int)sizeof(int) + 15) & ~15));
        X.pwa = wb;
        X.pwb = wb + nf;
        X.xy = A.xf[l0 + q].xy;
        return X;
    };
    // Copy into LDS: the top level's r and sigma (all threads), one level's per-plane
    // coefficient tables and one level pair's transfer tables per wave.  Every load of the
    // first pass is issued before the first LDS store, so the copy costs one round trip to
    // memory; the later passes (levels with more than 64 planes, more than 8 levels, more
    // than 8 values per thread) follow.
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
    constexpr int kU = 8;
    const Lv<T, 1> G0 = gview(A.lv[l0]);
    const Lv<T, 3> L0 = lvl(0);
    const int n0 = G0.nx * G0.ny * G0.nz;
    const int ns0 = G0.nx * G0.ny * (G0.sig_hi - G0.sig_lo);
    T v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int c = threadIdx.x + u * blockDim.x;
        v[u] = c < n0 ? G0.r[c] : (c < n0 + ns0 ? G0.sig[c - n0] : T(0));
    }
    const bool tq = wave < nl, xq = wave + 1 < nl;
    T tv[4] = {T(0), T(0), T(0), T(0)};
    int tnz = 0;
    if (tq) {
        const Lv<T, 1> G = gview(A.lv[l0 + wave]);
        tnz = G.nz;
        if (lane < tnz) { tv[0] = G.cxy[lane]; tv[1] = G.czm[lane]; tv[2] = G.czp[lane]; tv[3] = G.dg[lane]; }
    }
    int xc[3] = {0, 0, 0}, xf[3] = {0, 0, 0};
    T xw[2] = {T(0), T(0)};
    int xnf = 0, xnc = 0;
    if (xq) {
        const Xv<T> G = xview(A.xf[l0 + wave]);
        xnf = A.lv[l0 + wave].nz;
        xnc = A.lv[l0 + wave + 1].nz;
        if (lane < xnc) { xc[0] = G.cks[lane]; xc[1] = G.ccnt[lane]; xc[2] = G.cthick[lane]; }
        if (lane < xnf) {
            xf[0] = G.fthick[lane]; xf[1] = G.pka[lane]; xf[2] = G.pkb[lane];
            xw[0] = G.pwa[lane]; xw[1] = G.pwb[lane];
        }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int c = threadIdx.x + u * blockDim.x;
        if (c < n0) L0.r[c] = v[u];
        else if (c < n0 + ns0) L0.sig[c - n0] = v[u];
    }
    if (tq && lane < tnz) {
        T FX_AS(3) *tab = (T FX_AS(3) *)(lds + A.off_t[wave]);
        tab[lane] = tv[0]; tab[tnz + lane] = tv[1]; tab[2 * tnz + lane] = tv[2]; tab[3 * tnz + lane] = tv[3];
    }
    if (xq) {
        const Xv<T, 3> X = xlds(wave);
        int FX_AS(3) *ib = (int FX_AS(3) *)X.cks;
        T FX_AS(3) *wb = (T FX_AS(3) *)X.pwa;
        if (lane < xnc) { ib[lane] = xc[0]; ib[xnc + lane] = xc[1]; ib[2 * xnc + lane] = xc[2]; }
        if (lane < xnf) {
            ib[3 * xnc + lane] = xf[0]; ib[3 * xnc + xnf + lane] = xf[1]; ib[3 * xnc + 2 * xnf + lane] = xf[2];
            wb[lane] = xw[0]; wb[xnf + lane] = xw[1];
        }
    }
    for (int c = threadIdx.x + kU * blockDim.x; c < n0 + ns0; c += blockDim.x) {
        if (c < n0) L0.r[c] = G0.r[c];
        else L0.sig[c - n0] = G0.sig[c - n0];
    }
    for (int q = wave; q < nl; q += nwave) {
        const Lv<T, 1> G = gview(A.lv[l0 + q]);
        T FX_AS(3) *tab = (T FX_AS(3) *)(lds + A.off_t[q]);
        for (int c = (q == wave ? 64 : 0) + lane; c < G.nz; c += 64) {
            tab[c] = G.cxy[c];
            tab[G.nz + c] = G.czm[c];
            tab[2 * G.nz + c] = G.czp[c];
            tab[3 * G.nz + c] = G.dg[c];
        }
    }
    for (int q = wave; q + 1 < nl; q += nwave) {
        const Xv<T> G = xview(A.xf[l0 + q]);
        const int nf = A.lv[l0 + q].nz, nc = A.lv[l0 + q + 1].nz;
        const Xv<T, 3> X = xlds(q);
        int FX_AS(3) *ib = (int FX_AS(3) *)X.cks;
        T FX_AS(3) *wb = (T FX_AS(3) *)X.pwa;
        const int c0 = q == wave ? 64 : 0;
        for (int c = c0 + lane; c < nc; c += 64) {
            ib[c] = G.cks[c];
            ib[nc + c] = G.ccnt[c];
            ib[2 * nc + c] = G.cthick[c];
        }
        for (int c = c0 + lane; c < nf; c += 64) {
            ib[3 * nc + c] = G.fthick[c];
            ib[3 * nc + nf + c] = G.pka[c];
            ib[3 * nc + 2 * nf + c] = G.pkb[c];
            wb[c] = G.pwa[c];
            wb[nf + c] = G.pwb[c];
        }
    }
    __syncthreads();
    // levels qw.. and the bottom fit one wave (qw = nl: the bottom does not)
    for (int q = 0; q < min(qw, nl - 1); ++q) co_down<0>(lvl(q), lvl(q + 1), xlds(q), nu1);
    if (qw >= nl) {
        const Lv<T, 3> B = lvl(nl - 1);
        T FX_AS(3) *rs = (T FX_AS(3) *)(lds + A.off_p);
        double FX_AS(3) *red = (double FX_AS(3) *)(lds + A.off_red);     // more than 64 cells: room for 32
        bottom_block<T>(B, rs, red, A.bottom_iters, A.bottom_tol2);
    } else {
        if (threadIdx.x < 64) {
            for (int q = qw; q < nl - 1; ++q) co_down<1>(lvl(q), lvl(q + 1), xlds(q), nu1);
            bottom_wave<T>(lvl(nl - 1), A.bottom_iters, A.bottom_tol2);
            Crew<1>::sync();
            for (int q = nl - 2; q >= qw; --q) co_up<1>(lvl(q), lvl(q + 1), xlds(q), nu2);
        }
        __syncthreads();
    }
    for (int q = min(qw, nl - 1) - 1; q >= 0; --q) co_up<0>(lvl(q), lvl(q + 1), xlds(q), nu2);
    {
        const Lv<T, 1> G = gview(A.lv[l0]);
        const Lv<T, 3> L0 = lvl(0);
        const int n = G.nx * G.ny * G.nz;
        for (int c = threadIdx.x; c < n; c += blockDim.x) G.e[c] = L0.e[c];
    }
}

// Start of a run (or of one chunk of its schedule): nsteps more time steps.
// first = 0 keeps instances whose solve failed in an earlier chunk parked.
template <typename T>
__global__ void k_run_setup(const Inst<T> *I, int ninst, int nsteps, int has_sched, double dt, int first) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= ninst) return;
    GState *s = asp<1>(I[n].st);
    const bool failed = !first && s->status != 0;
    if (first) { s->status = 0; s->max_cycles_step = 0; }
    s->target = s->step + nsteps;
    s->sched_base = s->step;
    s->sched_len = has_sched ? nsteps : 0;
    s->dt = dt;
    s->parked = nsteps == 0 || failed;
    s->adv = 0;
}

template <typename T>
__global__ void k_set_vtop(const Inst<T> *I, int ninst, double v) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n < ninst) asp<1>(I[n].st)->v_top = v;
}

__global__ void k_put_state(InstState *dst, InstState v) {
    if (threadIdx.x == 0) *dst = v;
}

__global__ void k_zero32(unsigned *x, size_t n) {
    for (size_t c = blockIdx.x * (size_t)blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x) x[c] = 0u;
}

__global__ void k_fill(double *x, size_t n, double v) {
    for (size_t c = blockIdx.x * (size_t)blockDim.x + threadIdx.x; c < n; c += (size_t)gridDim.x * blockDim.x) x[c] = v;
}

}  // namespace

// ------------------------------------------------------------------ launchers
#define FX_LAUNCH(kern, w, ...)                                                                            \
    do {                                                                                                   \
        if ((w).total > 0) hipLaunchKernelGGL(kern, grid_of((w).total), dim3(BX, BY), 0, st, __VA_ARGS__); \
    } while (0)

template <typename T>
void launch_tdgl(const Inst<T> *I, const Work &w, hipStream_t st) {
    FX_LAUNCH(k_tdgl<T>, w, I, w);
}

// One launch on small problems, where a launch costs more than its work; from about 2^21 device
// cells two, each with its own register budget (shared, the TDGL tiles run at the
// extrapolation's lower occupancy: 256 x 256 x 120 cells took 84 us together and 75 us apart,
// 128 x 128 x 48 cells 8.3 us together and 11.1 us apart).
template <typename T>
void launch_fields(const Inst<T> *I, const Work &wt, const Work &we, int rec, hipStream_t st) {
    const int gt = wt.total > 0 ? (int)grid_of(wt.total).x : 0, ge = (int)grid_of(we.total).x;
    const int gq = rec ? wt.ninst * kQvBlocks : 0;
    if (we.total < (1 << 21) / kExtrapChunk) {
        hipLaunchKernelGGL((k_fields<T, 3>), dim3(gt + ge + gq), dim3(BX, BY), 0, st, I, wt, we, gt, ge);
        return;
    }
    if (gt) hipLaunchKernelGGL((k_fields<T, 1>), dim3(gt), dim3(BX, BY), 0, st, I, wt, we, gt, 0);
    hipLaunchKernelGGL((k_fields<T, 2>), dim3(ge + gq), dim3(BX, BY), 0, st, I, wt, we, 0, ge);
}

inline dim3 per_inst(int ninst) { return dim3((ninst + 63) / 64); }

template <typename T>
void launch_qv(const Inst<T> *I, int ninst, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_qv_part<T>, dim3(ninst * kQvBlocks), dim3(256), 0, st, I);
    hipLaunchKernelGGL(k_qv_fin<T>, per_inst(ninst), dim3(64), 0, st, I, ninst, out);
}

template <typename T>
void launch_flip(const Inst<T> *I, int ninst, hipStream_t st) {
    hipLaunchKernelGGL(k_flip<T>, per_inst(ninst), dim3(64), 0, st, I, ninst);
}

template <typename T>
void launch_begin(const Inst<T> *I, InstState *S, int ninst, int sel, hipStream_t st) {
    hipLaunchKernelGGL(k_begin<T>, per_inst(ninst), dim3(64), 0, st, I, S, ninst, sel);
}

template <typename T>
void launch_residual(const Inst<T> *I, const ResWork &w, int after_cycle, int any_fd, hipStream_t st) {
    auto *k0 = any_fd ? &k_residual<T, 0, 1> : &k_residual<T, 0, 0>;
    auto *k2 = any_fd ? &k_residual<T, 2, 1> : &k_residual<T, 2, 0>;
    FX_LAUNCH(k0, w.cell0, I, w.cell0, after_cycle);
    if (after_cycle) FX_LAUNCH(k2, w.cell2, I, w.cell2, after_cycle);
}

template <typename T>
void launch_reduce(const Inst<T> *I, InstState *S, int ninst, int mode, int rec, hipStream_t st) {
    auto *k = mode == 2 ? &k_reduce<T, 2> : mode == 1 ? &k_reduce<T, 1> : &k_reduce<T, 0>;
    hipLaunchKernelGGL(k, dim3(ninst), dim3(1024), 0, st, I, S, rec);
}

template <typename T, int ZT>
struct SmoothSet {
    template <typename F>
    static void pick(int upd, int zero_init, int w8, F go) {
        if (w8) {
            if (upd) go(k_smooth_w8<T, 0, ZT, 1>);
            else if (zero_init) go(k_smooth_w8<T, 1, ZT, 0>);
            else go(k_smooth_w8<T, 0, ZT, 0>);
        } else {
            if (upd) go(k_smooth<T, 0, ZT, 1>);
            else if (zero_init) go(k_smooth<T, 1, ZT, 0>);
            else go(k_smooth<T, 0, ZT, 0>);
        }
    }
};

template <typename T>
void launch_smooth(const Inst<T> *I, const Work &w, int level, int color, int zero_init, int upd, const SmoothCfg &c,
                   double *probe, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, int skip_light) {
    if (w.total <= 0) return;
    const dim3 g = grid_of(w.total);
    const int lbx = c.lbx;
    auto go = [&](auto kern) {
        if (ev0) hipExtLaunchKernelGGL(kern, g, dim3(256), 0, st, ev0, ev1, 0, I, w, level, color, lbx, probe, skip_light);
        else hipLaunchKernelGGL(kern, g, dim3(256), 0, st, I, w, level, color, lbx, probe, skip_light);
    };
    switch (c.zt) {
        case 8: SmoothSet<T, 8>::pick(upd, zero_init, c.w8, go); break;
        case 4: SmoothSet<T, 4>::pick(upd, zero_init, c.w8, go); break;
        case 2: SmoothSet<T, 2>::pick(upd, zero_init, c.w8, go); break;
        default: SmoothSet<T, 1>::pick(upd, zero_init, c.w8, go); break;
    }
}

template <typename T>
void launch_smooth_zpair(const Inst<T> *I, const Work &w, int level, const SmoothCfg &c, hipStream_t st) {
    if (w.total <= 0) return;
    const dim3 g = grid_of(w.total);
    switch (c.zt) {
        case 8: hipLaunchKernelGGL((k_smooth_zpair<T, 8>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
        case 4: hipLaunchKernelGGL((k_smooth_zpair<T, 4>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
        case 2: hipLaunchKernelGGL((k_smooth_zpair<T, 2>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
        default: hipLaunchKernelGGL((k_smooth_zpair<T, 1>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
    }
}

template <typename T>
void launch_prolong_red(const Inst<T> *I, const Work &w, int level, const SmoothCfg &c, hipStream_t st) {
    if (w.total <= 0) return;
    const dim3 g = grid_of(w.total);
    switch (c.zt) {
        case 8: hipLaunchKernelGGL((k_prolong_red<T, 8>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
        case 4: hipLaunchKernelGGL((k_prolong_red<T, 4>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
        case 2: hipLaunchKernelGGL((k_prolong_red<T, 2>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
        default: hipLaunchKernelGGL((k_prolong_red<T, 1>), g, dim3(256), 0, st, I, w, level, c.lbx); break;
    }
}

template <typename T>
void launch_restrict(const Inst<T> *I, const Work &w, int level, hipStream_t st) {
    FX_LAUNCH(k_restrict<T>, w, I, w, level);
}

template <typename T>
void launch_prolong(const Inst<T> *I, const Work &w, int level, hipStream_t st) {
    FX_LAUNCH(k_prolong<T>, w, I, w, level);
}

template <typename T>
void launch_prolong_cc(const Inst<T> *I, const Work &w, int level, int cz, hipStream_t st) {
    FX_LAUNCH(k_prolong_cc<T>, w, I, w, level, cz);
}

template <typename T>
void launch_pre_tb(const Inst<T> *I, const Work &w, int level, int nu, int nz, hipStream_t st) {
    if (w.total <= 0) return;
    const size_t lds = tb_lds_bytes(nz, 0, sizeof(T));
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid_of(w.total), dim3(kTbThreads), lds, st, I, w, level, nu); };
    switch (tb_zq(nz)) {
        case 1: go(k_pre_tb<T, 1>); break;
        case 2: go(k_pre_tb<T, 2>); break;
        case 3: go(k_pre_tb<T, 3>); break;
        case 4: go(k_pre_tb<T, 4>); break;
        case 6: go(k_pre_tb<T, 6>); break;
        default: go(k_pre_tb<T, 8>); break;
    }
}
template <typename T, int FINEST>
static void launch_post_tb_f(const Inst<T> *I, const Work &w, int level, int nu, int nz, int nzc, hipStream_t st) {
    const size_t lds = tb_lds_bytes(nz, nzc, sizeof(T));
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid_of(w.total), dim3(kTbThreads), lds, st, I, w, level, nu); };
    switch (tb_zq(nz)) {
        case 1: go(k_post_tb<T, 1, FINEST>); break;
        case 2: go(k_post_tb<T, 2, FINEST>); break;
        case 3: go(k_post_tb<T, 3, FINEST>); break;
        case 4: go(k_post_tb<T, 4, FINEST>); break;
        case 6: go(k_post_tb<T, 6, FINEST>); break;
        default: go(k_post_tb<T, 8, FINEST>); break;
    }
}
template <typename T>
void launch_post_tb(const Inst<T> *I, const Work &w, int level, int nu, int nz, int nzc, hipStream_t st) {
    if (w.total <= 0) return;
    if (level == 0) launch_post_tb_f<T, 1>(I, w, level, nu, nz, nzc, st);
    else launch_post_tb_f<T, 0>(I, w, level, nu, nz, nzc, st);
}
template <typename T>
void launch_pre_zm(const Inst<T> *I, const Work &w, int level, int nu, int zl, hipStream_t st) {
    if (w.total <= 0) return;
    hipLaunchKernelGGL(k_pre_zm<T>, grid_of(w.total), dim3(kZmThreads), zm_lds_bytes(zl, 0, sizeof(T)), st, I, w, level, nu, zl);
}
template <typename T>
void launch_post_zm(const Inst<T> *I, const Work &w, int level, int nu, int zl, hipStream_t st) {
    if (w.total <= 0) return;
    const size_t lds = zm_lds_bytes(zl, 1, sizeof(T));
    if (level == 0) hipLaunchKernelGGL((k_post_zm<T, 1>), grid_of(w.total), dim3(kZmThreads), lds, st, I, w, level, nu, zl);
    else hipLaunchKernelGGL((k_post_zm<T, 0>), grid_of(w.total), dim3(kZmThreads), lds, st, I, w, level, nu, zl);
}
template <typename T>
void launch_coarse(const Inst<T> *I, InstState *S, int ninst, int lds_bytes, hipStream_t st) {
    hipLaunchKernelGGL(k_coarse<T>, dim3(ninst), dim3(kCoarseThreads), lds_bytes, st, I, S);
}

template <typename T>
void launch_head(const Inst<T> *I, InstState *S, int ninst, int advance, hipStream_t st) {
    hipLaunchKernelGGL(k_head<T>, per_inst(ninst), dim3(64), 0, st, I, S, ninst, advance);
}


template <typename T>
void launch_run_setup(const Inst<T> *I, int ninst, int nsteps, int has_sched, double dt, int first, hipStream_t st) {
    hipLaunchKernelGGL(k_run_setup<T>, per_inst(ninst), dim3(64), 0, st, I, ninst, nsteps, has_sched, dt, first);
}

template <typename T>
void launch_set_vtop(const Inst<T> *I, int ninst, double v, hipStream_t st) {
    hipLaunchKernelGGL(k_set_vtop<T>, per_inst(ninst), dim3(64), 0, st, I, ninst, v);
}

void launch_put_state(InstState *dst, const InstState &v, hipStream_t st) {
    hipLaunchKernelGGL(k_put_state, dim3(1), dim3(64), 0, st, dst, v);
}

void launch_zero(void *x, size_t bytes, hipStream_t st) {
    const size_t n = bytes / 4, b = (n + 255) / 256;
    hipLaunchKernelGGL(k_zero32, dim3(b == 0 ? 1 : (b < 4096 ? (unsigned)b : 4096u)), dim3(256), 0, st, (unsigned *)x, n);
}

void launch_fill(double *x, size_t n, double v, hipStream_t st) {
    const size_t b = (n + 255) / 256;
    hipLaunchKernelGGL(k_fill, dim3(b == 0 ? 1 : (b < 4096 ? (unsigned)b : 4096u)), dim3(256), 0, st, x, n, v);
}

#define FX_INST(T)                                                                                           \
    template void launch_tdgl<T>(const Inst<T> *, const Work &, hipStream_t);                                \
    template void launch_fields<T>(const Inst<T> *, const Work &, const Work &, int, hipStream_t);           \
    template void launch_flip<T>(const Inst<T> *, int, hipStream_t);                                        \
    template void launch_qv<T>(const Inst<T> *, int, double *, hipStream_t);                                 \
    template void launch_begin<T>(const Inst<T> *, InstState *, int, int, hipStream_t);                                  \
    template void launch_residual<T>(const Inst<T> *, const ResWork &, int, int, hipStream_t);                    \
    template void launch_reduce<T>(const Inst<T> *, InstState *, int, int, int, hipStream_t);                \
    template void launch_smooth<T>(const Inst<T> *, const Work &, int, int, int, int, const SmoothCfg &,     \
                                   double *, hipStream_t, hipEvent_t, hipEvent_t, int);                      \
    template void launch_smooth_zpair<T>(const Inst<T> *, const Work &, int, const SmoothCfg &, hipStream_t); \
    template void launch_prolong_red<T>(const Inst<T> *, const Work &, int, const SmoothCfg &, hipStream_t);  \
    template void launch_restrict<T>(const Inst<T> *, const Work &, int, hipStream_t);                       \
    template void launch_prolong<T>(const Inst<T> *, const Work &, int, hipStream_t);                        \
    template void launch_prolong_cc<T>(const Inst<T> *, const Work &, int, int, hipStream_t);                \
    template void launch_coarse<T>(const Inst<T> *, InstState *, int, int, hipStream_t);                      \
    template void launch_pre_tb<T>(const Inst<T> *, const Work &, int, int, int, hipStream_t);                \
    template void launch_post_tb<T>(const Inst<T> *, const Work &, int, int, int, int, hipStream_t);          \
    template void launch_pre_zm<T>(const Inst<T> *, const Work &, int, int, int, hipStream_t);                \
    template void launch_post_zm<T>(const Inst<T> *, const Work &, int, int, int, hipStream_t);               \
    template void launch_head<T>(const Inst<T> *, InstState *, int, int, hipStream_t);                                    \
    template void launch_run_setup<T>(const Inst<T> *, int, int, int, double, int, hipStream_t);             \
    template void launch_set_vtop<T>(const Inst<T> *, int, double, hipStream_t);
FX_INST(double)
FX_INST(float)

}  // namespace fx
