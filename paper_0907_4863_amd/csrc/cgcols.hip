// Level-0 passes with one stencil, by columns (cols.h): the two passes of a CG step, the true
// residual, and the step of the Lanczos estimate.
//
// A wavefront marches 3 lines of 62 columns (lanes 0 and 63 are the halo) along z and loads
// the lines before and after them itself, so that wavefronts share nothing and no plane takes a
// barrier; the four wavefronts of a block take consecutive lines, whose halo lines they find in
// the cache.  An operand's plane is loaded one plane ahead and its values are formed when the
// plane arrives, one plane before they are the centre of the stencil.
//
// A CG step in this form keeps no q = A p: the first pass forms the new direction at the stencil's
// nodes from z and the old one and sums p . A p, the second forms A p again for r -= alpha A p, in
// fp64 throughout.  Per unknown 36 + 28 bytes in mixed precision against 52 + 28 with q.  On the
// 145 x 145 x 435 ellipse the passes move 360 and 270 MB (rows that start off the cache lines
// are written in 27% more than their bytes) at 4.5 and 4 TB/s.
#include "cols.h"

namespace saamg {

constexpr int kColThreads = 256;

// A lane's nodes in a plane, as byte offsets of values of 4 and 8 bytes: the 5 lines (own 1..3)
// a pass loads, and the 3 it writes.
struct ColAt {
    unsigned l4[5], l8[5], s4[3], s8[3];
    template <typename E>
    __device__ __forceinline__ unsigned ld(int k) const { return sizeof(E) == 4 ? l4[k] : l8[k]; }
    template <typename E>
    __device__ __forceinline__ unsigned st(int k) const { return sizeof(E) == 4 ? s4[k] : s8[k]; }
};

// March of a wavefront: for every plane the op loads (op.load), forms its 5 values
// (op.form(line)) and writes what needs no stencil (op.emit), then op.body(l, c, ax) takes the
// centre and A X of the own lines.
template <bool SP = false, class Op>
__device__ __forceinline__ void col_march(const StrokeView<double>& v, Op& op) {
    int tx, ty, sz;
    stroke_tile(v, &tx, &ty, &sz);
    const int lane = threadIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int x = kColX * tx - 1 + lane, yb = kColLines * ty + 3 * w;
    const int zs = sz * v.S, ze = min(zs + v.S, v.nz);
    if (yb >= v.ny) return;
    ColAt at;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int y = yb + k - 1;
        const bool in = (unsigned)x < (unsigned)v.nx && (unsigned)y < (unsigned)v.ny;
        const unsigned o = (unsigned)(v.nx * y + x);
        at.l4[k] = in ? 4u * o : kOff;
        at.l8[k] = in ? 8u * o : kOff;
        if (k >= 1 && k <= 3) {
            const bool own = in && lane >= 1 && lane <= kColX;
            at.s4[k - 1] = own ? 4u * o : kOff;
            at.s8[k - 1] = own ? 8u * o : kOff;
        }
    }
    Rows<double, false, SP> rows;
    rows.init(v, yb, zs);
    op.start(v.nxy, zs - 1);
    op.load(at, zs >= 1);
    double V[3][3], H[2][2];  // the own lines on three planes; the lines beside them on two
#pragma unroll
    for (int l = 0; l < 3; ++l) V[0][l] = V[1][l] = V[2][l] = 0.0;
    H[0][0] = H[0][1] = H[1][0] = H[1][1] = 0.0;
    // plane p is the centre; the plane above it has been loaded
    auto step = [&](auto ph, int p) {
        constexpr int A = decltype(ph)::value, B = (A + 2) % 3, C = (A + 1) % 3;
        H[0][0] = H[1][0];
        H[0][1] = H[1][1];
        H[1][0] = op.form(0);
        H[1][1] = op.form(4);
#pragma unroll
        for (int l = 0; l < 3; ++l) V[C][l] = op.form(l + 1);
        op.emit(at, p + 1 >= zs && p + 1 < ze);
        op.load(at, p + 2 < v.nz && p + 2 <= ze);
        if (p >= zs && rows.next(v, x, yb, zs, p - zs)) {
            double ax[3];
            apply3<double>(rows.c.a, V[A], V[B], V[C], H[0][0], H[0][1], ax);
#pragma unroll
            for (int l = 0; l < 3; ++l) op.body(at, l, V[A][l], ax[l]);
        }
        op.next();
    };
    for (int p = zs - 2; p < ze; p += 3) {
        step(std::integral_constant<int, 0>{}, p);
        if (p + 1 < ze) step(std::integral_constant<int, 1>{}, p + 1);
        if (p + 2 < ze) step(std::integral_constant<int, 2>{}, p + 2);
    }
}

// The next CG direction pn = z + beta p and the partials of pn . A pn; on the way x += xa p, the
// update the previous step still owes x.
template <typename TZ>
struct DirOp {
    const TZ* z;
    const double* p;
    double* pn;
    double* x;
    int b4, b8;  // bytes of a plane
    double beta, xa;
    double acc = 0.0;
    TZ rz[5];
    double rp[5], rx[3], val[5];
    long nxy;
    __device__ __forceinline__ void start(long nxy_, int zp) {
        nxy = nxy_;
        z += nxy * zp;
        p += nxy * zp;
        pn += nxy * zp;
        x += nxy * zp;
    }
    __device__ __forceinline__ void load(const ColAt& at, bool ok) {
        const auto bz = plane(z, sizeof(TZ) == 4 ? b4 : b8, ok), bp = plane(p, b8, ok);
#pragma unroll
        for (int l = 0; l < 5; ++l) {
            bload(bz, at.ld<TZ>(l), rz[l]);
            bload(bp, at.l8[l], rp[l]);
        }
        z += nxy;
        p += nxy;
        const auto bx = plane(x, b8, ok);
#pragma unroll
        for (int l = 0; l < 3; ++l) bload(bx, at.s8[l], rx[l]);
    }
    __device__ __forceinline__ double form(int l) {
        rz[l] = here(rz[l]);
        rp[l] = here(rp[l]);
        return val[l] = __builtin_fma(beta, rp[l], (double)rz[l]);
    }
    __device__ __forceinline__ void emit(const ColAt& at, bool ok) {
        const auto bn = plane((const double*)pn, b8, ok), bx = plane((const double*)x, b8, ok);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            bstore(bn, at.s8[l], val[l + 1]);
            bstore(bx, at.s8[l], __builtin_fma(xa, rp[l + 1], here(rx[l])));
        }
        pn += nxy;
        x += nxy;
    }
    __device__ __forceinline__ void body(const ColAt& at, int l, double c, double ax) {
        acc += at.s8[l] != kOff ? c * ax : 0.0;
    }
    __device__ __forceinline__ void next() {}
};

template <typename TZ>
__global__ void __launch_bounds__(kColThreads) k_col_dir(StrokeView<double> v, const TZ* __restrict__ z,
                                                         const double* __restrict__ p,
                                                         double* __restrict__ pn, double* __restrict__ x,
                                                         const double* __restrict__ scal, double* part) {
    __shared__ double lds[kColThreads / kWave];
    DirOp<TZ> op;
    op.z = z;
    op.p = p;
    op.pn = pn;
    op.x = x;
    op.b4 = (int)(4 * v.nxy);
    op.b8 = (int)(8 * v.nxy);
    op.beta = scal[S_BETA];
    op.xa = scal[S_XA];
    col_march(v, op);
    const double s = block_sum(op.acc, lds);
    if (threadIdx.x == 0 && threadIdx.y == 0) part[blockIdx.x] = s;
}

// r -= alpha A p (alpha = S_XA; r left as it is when the step broke down), its fp32 copy (mixed
// precision) and the partials of r . r.
template <bool MIX>
struct ResOp {
    const double* p;
    double* r;
    float* r32;
    int b4, b8;
    double alpha;
    double acc = 0.0;
    double rp[5], rr[3], cur[3];
    long nxy;
    __device__ __forceinline__ void start(long nxy_, int zp) {
        nxy = nxy_;
        p += nxy * zp;
        r += nxy * zp;
        if (MIX) r32 += nxy * zp;
#pragma unroll
        for (int l = 0; l < 3; ++l) rr[l] = cur[l] = 0.0;
    }
    // p of the next plane up, and r one plane behind it (loaded when p of that plane is formed)
    __device__ __forceinline__ void load(const ColAt& at, bool ok) {
        const auto bp = plane(p, b8, ok);
#pragma unroll
        for (int l = 0; l < 5; ++l) bload(bp, at.l8[l], rp[l]);
        p += nxy;
    }
    __device__ __forceinline__ double form(int l) { return rp[l] = here(rp[l]); }
    __device__ __forceinline__ void emit(const ColAt& at, bool ok) {
        // r of the plane just formed, used when it is the centre
#pragma unroll
        for (int l = 0; l < 3; ++l) cur[l] = here(rr[l]);
        const auto b = plane((const double*)r, b8, ok);
#pragma unroll
        for (int l = 0; l < 3; ++l) bload(b, at.s8[l], rr[l]);
    }
    __device__ __forceinline__ void body(const ColAt& at, int l, double, double ax) {
        const double o = alpha != 0.0 ? cur[l] - alpha * ax : cur[l];
        if (alpha != 0.0) {
            bstore(plane((const double*)(r - nxy), b8, true), at.s8[l], o);
            if (MIX) bstore(plane((const float*)(r32 - nxy), b4, true), at.s4[l], (float)o);
        }
        acc += at.s8[l] != kOff ? o * o : 0.0;
    }
    __device__ __forceinline__ void next() {
        r += nxy;
        if (MIX) r32 += nxy;
    }
};

template <bool MIX>
__global__ void __launch_bounds__(kColThreads) k_col_res(StrokeView<double> v,
                                                         const double* __restrict__ p,
                                                         double* __restrict__ r,
                                                         float* __restrict__ r32,
                                                         const double* __restrict__ scal, double* part) {
    __shared__ double lds[kColThreads / kWave];
    ResOp<MIX> op;
    op.p = p;
    op.r = r;
    op.r32 = r32;
    op.b4 = (int)(4 * v.nxy);
    op.b8 = (int)(8 * v.nxy);
    op.alpha = scal[S_XA];
    col_march(v, op);
    const double s = block_sum(op.acc, lds);
    if (threadIdx.x == 0 && threadIdx.y == 0) part[blockIdx.x] = s;
}

// The true residual r = bs - A x with its fp32 copy (r32 not null), and the partials of r.r and
// bs.bs.  FLUSH: of x' = x + xa p, the update that the last step still owes x, written to xn (the
// neighbours still read x).
template <bool FLUSH>
struct ResidOp {
    const double *x, *p, *bs;
    double *xn, *r;
    float* r32;
    int b4, b8;
    double xa;
    double rr = 0.0, bb = 0.0;
    double rx[5], rp[5], rb[3], cur[3], val[5];
    long nxy;
    __device__ __forceinline__ void start(long nxy_, int zp) {
        nxy = nxy_;
        x += nxy * zp;
        bs += nxy * zp;
        r += nxy * zp;
        if (FLUSH) {
            p += nxy * zp;
            xn += nxy * zp;
        }
        if (r32) r32 += nxy * zp;
#pragma unroll
        for (int l = 0; l < 3; ++l) rb[l] = cur[l] = 0.0;
    }
    __device__ __forceinline__ void load(const ColAt& at, bool ok) {
        const auto bx = plane(x, b8, ok), bp = plane(FLUSH ? p : x, b8, ok);
#pragma unroll
        for (int l = 0; l < 5; ++l) {
            bload(bx, at.l8[l], rx[l]);
            if (FLUSH) bload(bp, at.l8[l], rp[l]);
        }
        x += nxy;
        if (FLUSH) p += nxy;
    }
    __device__ __forceinline__ double form(int l) {
        rx[l] = here(rx[l]);
        return val[l] = FLUSH ? __builtin_fma(xa, here(rp[l]), rx[l]) : rx[l];
    }
    __device__ __forceinline__ void emit(const ColAt& at, bool ok) {
        // bs of the plane just formed, used when it is the centre
        const auto b = plane(bs, b8, ok);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            cur[l] = here(rb[l]);
            bload(b, at.s8[l], rb[l]);
        }
        if (FLUSH) {
            const auto bn = plane((const double*)xn, b8, ok);
#pragma unroll
            for (int l = 0; l < 3; ++l) bstore(bn, at.s8[l], val[l + 1]);
            xn += nxy;
        }
    }
    __device__ __forceinline__ void body(const ColAt& at, int l, double, double ax) {
        const double o = cur[l] - ax;
        bstore(plane((const double*)(r - nxy), b8, true), at.s8[l], o);
        if (r32) bstore(plane((const float*)(r32 - nxy), b4, true), at.s4[l], (float)o);
        const bool own = at.s8[l] != kOff;
        rr += own ? o * o : 0.0;
        bb += own ? cur[l] * cur[l] : 0.0;
    }
    __device__ __forceinline__ void next() {
        bs += nxy;
        r += nxy;
        if (r32) r32 += nxy;
    }
};

template <bool FLUSH>
__global__ void __launch_bounds__(kColThreads) k_col_resid(StrokeView<double> v, const double* __restrict__ bs,
                                                           const double* __restrict__ x,
                                                           const double* __restrict__ p,
                                                           double* __restrict__ xn, double* __restrict__ r,
                                                           float* __restrict__ r32,
                                                           const double* __restrict__ scal, double* part) {
    __shared__ double lds[kColThreads / kWave];
    ResidOp<FLUSH> op;
    op.x = x;
    op.p = p;
    op.bs = bs;
    op.xn = xn;
    op.r = r;
    op.r32 = r32;
    op.b4 = (int)(4 * v.nxy);
    op.b8 = (int)(8 * v.nxy);
    op.xa = FLUSH ? scal[S_XA] : 0.0;
    col_march(v, op);
    const double s0 = block_sum(op.rr, lds), s1 = block_sum(op.bb, lds);
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        part[blockIdx.x] = s0;
        part[gridDim.x + blockIdx.x] = s1;
    }
}

// A step of the Lanczos recurrence in one pass: y' = cu u - cc y - cp w, with u = S y and w
// the vector before y, and u' = S y' for the next step; partials of y' . S y' and y' . y'.
// S is the symmetric part of A (SP: A itself is not symmetric), the vectors are kept as they
// come, and the scalars carry the norms (FIN_LZ).
struct LzOp {
    const double *u, *y, *w;
    double *yn, *un;
    int b8;
    double cu, cc, cp;
    double ya = 0.0, yy = 0.0;
    double ru[5], ry[5], rw[5], val[5];
    long nxy;
    __device__ __forceinline__ void start(long nxy_, int zp) {
        nxy = nxy_;
        u += nxy * zp;
        y += nxy * zp;
        w += nxy * zp;
        yn += nxy * zp;
        un += nxy * (zp - 1);
    }
    __device__ __forceinline__ void load(const ColAt& at, bool ok) {
        const auto bu = plane(u, b8, ok), by = plane(y, b8, ok), bw = plane(w, b8, ok);
#pragma unroll
        for (int l = 0; l < 5; ++l) {
            bload(bu, at.l8[l], ru[l]);
            bload(by, at.l8[l], ry[l]);
            bload(bw, at.l8[l], rw[l]);
        }
        u += nxy;
        y += nxy;
        w += nxy;
    }
    __device__ __forceinline__ double form(int l) {
        return val[l] = __builtin_fma(-cp, here(rw[l]), __builtin_fma(-cc, here(ry[l]), cu * here(ru[l])));
    }
    __device__ __forceinline__ void emit(const ColAt& at, bool ok) {
        const auto b = plane((const double*)yn, b8, ok);
#pragma unroll
        for (int l = 0; l < 3; ++l) bstore(b, at.s8[l], val[l + 1]);
        yn += nxy;
    }
    __device__ __forceinline__ void body(const ColAt& at, int l, double c, double ax) {
        bstore(plane((const double*)un, b8, true), at.s8[l], ax);
        const bool own = at.s8[l] != kOff;
        ya += own ? c * ax : 0.0;
        yy += own ? c * c : 0.0;
    }
    __device__ __forceinline__ void next() { un += nxy; }
};

// Bound by its 40 bytes a node.  With u = S v in a pass of its own and the update and its norm in
// another it was 48 bytes, in marches that read masks and slots per plane (see l0_lz_cols).
template <bool SP>
__global__ void __launch_bounds__(kColThreads) k_col_lz(StrokeView<double> v, const double* __restrict__ u,
                                                        const double* __restrict__ y,
                                                        const double* __restrict__ w,
                                                        double* __restrict__ yn, double* __restrict__ un,
                                                        const double* __restrict__ scal, double* part) {
    __shared__ double lds[kColThreads / kWave];
    LzOp op;
    op.u = u;
    op.y = y;
    op.w = w;
    op.yn = yn;
    op.un = un;
    op.b8 = (int)(8 * v.nxy);
    op.cu = scal[S_LZ_S];
    op.cc = scal[S_ALPHA];
    op.cp = scal[S_LZ_B];
    col_march<SP>(v, op);
    const double s0 = block_sum(op.ya, lds), s1 = block_sum(op.yy, lds);
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        part[blockIdx.x] = s0;
        part[gridDim.x + blockIdx.x] = s1;
    }
}

// Whether the CG passes of a box on one-node lanes run by columns: from 600 thousand unknowns on
// (the wavefront's start, from its tile to its rows, is four dependent loads), and where a
// plane is within a 32-bit byte offset.  The two passes against the fused q-recursion and its
// r update (fine.hip), which stay below: 97 x 97 x 291 cavity (0.9 million unknowns) 59 -> 46
// us, 128 x 128 x 256 ellipse 78 -> 57 us, mixed the same, 145 x 145 x 435 ellipse 218 -> 146 us;
// 64 x 64 x 128 cylinder (0.4 million) 15 -> 20 us, 33^3 9 -> 14 us.  Near the line whole solves
// take, without over with columns, 0.99 (97^3 cylinder, 0.7 million), 1.03 (80 x 80 x 160, 0.8 million)
// and 1.03 (112^3, 1.1 million), in both precisions.  On the 16-byte lanes of
// wide.hip the passes were faster than by columns (256 x 256 x 768, fp32 direction: 138 + 227
// us against 153 + 246).
//
// Where lines change along z (see l0_strokes) the rows read again cost more than masks and slots
// per plane (solves without / with columns): 80 x 80 x 160 straight 1.03, share 0.08 0.96; 97 x 97
// x 194 0.06 1.02, each plane 0.94; 128 x 128 x 256 0.16 1.01, each plane 0.92.  Long rows gain at any
// share on boxes of 1 to 3 million nodes (139^3, 257 x 60 x 130 and 291 x 97 x 97 with a change on
// each plane 1.04), on larger ones below 0.7 (145 x 145 x 290 0.53 1.03, each plane 0.95).
bool l0_cols_box(const FineLevel& L) {
    return !L.wide && L.n_unknowns >= 600000 && L.nxy * 8 < (long)kOff;
}
bool l0_cols(const FineLevel& L) {
    double most;
    if (L.nx > 128)
        most = L.nbox < 3000000 ? 1.0 : 0.7;
    else
        most = L.nbox < 2000000 ? 0.06 : 0.3;
    return l0_cols_box(L) && l0_change(L) <= most;
}
long l0_col_parts(const FineLevel& L) { return L.col.blocks(); }

static StrokeView<double> col_view(const FineLevel& L) {
    const L0View<double> l = L.view<double>();
    StrokeView<double> v;
    v.nx = L.nx; v.ny = L.ny; v.nz = L.nz; v.nsegx = L.nsegx; v.nxy = L.nxy;
    v.unk = l.unk; v.irr = l.irr; v.base = l.base; v.tab = l.tab; v.tabT = l.tabT;
    for (int a = 0; a < 3; ++a) v.c[a] = l.c[a];
    v.zinfo = L.zinfo;
    v.tiles = L.tiles + L.col.list;
    v.live = L.col.live;
    v.S = L.col.S;
    v.skip = nullptr;
    return v;
}

// Boxes on one-node lanes, where a plane is within a 32-bit byte offset: 145 x 145 x 435 ellipse
// 126 -> 103 us a step, 128 x 128 x 256 with quadratic rows 70 -> 44; 64 x 64 x 128 18 -> 15.  Boxes on
// 16-byte lanes keep their two passes (256 x 256 x 768: 15 steps 8.2 ms against 8.7 by columns), and
// so do small boxes whose lines change (33^3 cavity 0.80, with open ends 0.95; from 72^3 on 1.05
// and more).
bool l0_lz_cols(const FineLevel& L) {
    return !L.wide && L.nxy * 8 < (long)kOff && (L.nbox >= 350000 || l0_change(L) <= 0.045);
}

void col_lz(const FineLevel& L, bool sym, const double* u, const double* y, const double* w, double* yn,
            double* un, const double* scal, double* partials, hipStream_t s) {
    const dim3 g((unsigned)L.col.blocks()), b(kWave, 4);
    if (sym)
        hipLaunchKernelGGL(k_col_lz<false>, g, b, 0, s, col_view(L), u, y, w, yn, un, scal, partials);
    else
        hipLaunchKernelGGL(k_col_lz<true>, g, b, 0, s, col_view(L), u, y, w, yn, un, scal, partials);
    HIPCHECK(hipGetLastError());
}

void col_resid(const FineLevel& L, const double* bs, const double* x, const double* p, double* xn, double* r,
               float* r32, const double* scal, double* partials, hipStream_t s) {
    const dim3 g((unsigned)L.col.blocks()), b(kWave, 4);
    if (p)
        hipLaunchKernelGGL(k_col_resid<true>, g, b, 0, s, col_view(L), bs, x, p, xn, r, r32, scal, partials);
    else
        hipLaunchKernelGGL(k_col_resid<false>, g, b, 0, s, col_view(L), bs, x, p, xn, r, r32, scal, partials);
    HIPCHECK(hipGetLastError());
}

template <typename TZ>
void col_dir(const FineLevel& L, const TZ* z, double* x, const double* p, double* pn,
             const double* scal, double* partials, hipStream_t s) {
    KTimer kt(T_CG_PQ, s, L.n_unknowns * (long)(sizeof(TZ) + 32) + zinfo_bytes(L));
    klaunch(kt, true, k_col_dir<TZ>, dim3((unsigned)L.col.blocks()), dim3(kWave, 4), col_view(L), z,
            p, pn, x, scal, partials);
    HIPCHECK(hipGetLastError());
}
template void col_dir<float>(const FineLevel&, const float*, double*, const double*, double*,
                             const double*, double*, hipStream_t);
template void col_dir<double>(const FineLevel&, const double*, double*, const double*, double*,
                              const double*, double*, hipStream_t);

void col_res(const FineLevel& L, const double* p, double* r, float* r32, const double* scal,
             double* partials, hipStream_t s) {
    KTimer kt(T_CG_XR, s, L.n_unknowns * (24L + (r32 ? 4 : 0)) + zinfo_bytes(L));
    if (r32)
        klaunch(kt, true, k_col_res<true>, dim3((unsigned)L.col.blocks()), dim3(kWave, 4), col_view(L),
                p, r, r32, scal, partials);
    else
        klaunch(kt, true, k_col_res<false>, dim3((unsigned)L.col.blocks()), dim3(kWave, 4),
                col_view(L), p, r, r32, scal, partials);
    HIPCHECK(hipGetLastError());
}

}  // namespace saamg
