// Level-0 strokes of the V-cycle: the degree-2 pre-smoothing, the residual and the
// restriction in one pass over the lattice (down), and the prolongation with the degree-2
// post-smoothing and the PCG's r . z in one pass (up).
//
// A block of W wavefronts marches along z over a tile of lines.  A wavefront owns 64
// consecutive columns of 3 lines (one aggregate row), one column per lane and line, and
// the block's first and last wavefronts are the halo lines: a pass applies three stencils
// in a row, so the outputs lie 3 nodes inside the tile (2 for the up-stroke along x).
// The stages run as a pipeline along z: at plane p the first stage forms plane p - 1, the
// second p - 2, the third p - 3, each from the previous stage's three planes, which stay
// in registers.  x-neighbours come from the adjacent lanes, y-neighbours inside the three
// lines from registers; only the first and last line of each wavefront go through LDS,
// double-buffered, so that a plane takes one barrier.
//
// A column's stencil row (the six neighbour coefficients; zeros where the node is not an
// unknown) is held in registers and read again only where a line differs from the line one
// plane below (FineLevel::zinfo), which a pipe of constant cross-section does at its ends
// only: a plane then needs no masks, slots or table rows, and every lane runs the same
// code whether its row is regular, irregular or empty.
//
// Why one pass: the seven step kernels moved 20 + 4 and 28 bytes a node in fp32 where the
// strokes move 8 and 12, but each also paid a march's fixed cost per plane (masks, slots,
// table rows, 5 to 9 loads a node), and on small boxes a launch of 4-5 us.  On small boxes the
// strokes are bound by the latency of a plane step (0.45-0.6 us).  On the largest no unit is
// full: of 256 x 256 x 768 (fp32, down / up, counters) the vector units issue on 64 / 55% of the
// cycles of a busy compute unit (67 and 83 instructions an unknown, halo included), compute units
// are busy on 80% of the launch (480 blocks on 256 of them), 450 / 750 MB move at 3.6 / 4.1 TB/s
// where a copy of the same run moves 4.8, and a wavefront waits for loads or its plane's barrier
// on 54 / 59% of its cycles.  Time per V-cycle, step kernels -> down + up stroke:
//   256 x 256 x 768 ellipse, quadratic rule, fp32   612 -> 122 + 177 us
//   512^3 open tube, constant rule, fp32           1650 -> 308 + 455 us
//   128 x 128 x 256 ellipse, quadratic rule, fp64   223 ->  28 +  33 us
//   97 x 97 x 291 cavity with bore, fp32            118 ->  27 +  37 us
//   33^3 cylinder, fp64                              34 ->  10 +  12 us
#include <cstring>

#include "cols.h"

namespace saamg {

// Level 1 as the strokes address it.
template <typename T>
struct CoarseBox {
    int mx, my, mz;
    long sx, sxy;
    const T* invD;
};

// Barrier of a plane step: the LDS writes of the step are visible after it; loads and
// stores of device memory stay in flight.
__device__ __forceinline__ void step_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kStrokeMaxPlanes = 57;  // with its halo, a slab's planes fit the lanes of a wavefront
constexpr int kDownX = 57;  // columns of a down-stroke tile (19 aggregates)
constexpr int kUpX = 60;    // columns of an up-stroke tile

// x = the degree-2 Chebyshev iterate from zero; fc = P^T (f - A x), fd (nullable) = D^-1 fc.
template <typename T, bool SYM, int W>
__global__ void __launch_bounds__(64 * W) k_stroke_down(StrokeView<T> v, CoarseBox<T> cb,
                                                       const T* __restrict__ f,
                                                       T* __restrict__ xo, T* __restrict__ fc,
                                                       T* __restrict__ fd, T c1, T c2, T c20,
                                                       T omega) {
    __shared__ T sh[2][3][W + 2][2][64];
    __shared__ int ring[W][3][3][64];
    const double skip = v.skip ? *v.skip : 0.0;  // tested once the first loads are on their way
    int tx, ty, sz;
    stroke_tile(v, &tx, &ty, &sz);
    const int lane = threadIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int x = kDownX * tx - 3 + lane;
    const int yb = 3 * ((W - 2) * ty + w - 1);
    const int zs = sz * v.S, ze = min(zs + v.S, 3 * cb.mz);
    const int p0 = zs - 3;
    const bool own = w > 0 && w < W - 1;  // not a halo wavefront
    const bool useful = own && lane >= 3 && lane < 3 + kDownX;
    for (int i = lane + 64 * w; i < 2 * 3 * (W + 2) * 2 * 64; i += 64 * W) (&sh[0][0][0][0][0])[i] = T(0);

    Rows<T, !SYM> rows;
    rows.ring = &ring[w][0][0][0];
    rows.init(v, yb, p0);
    T F[3][3], X[3][3], R[3][3];
    T nf[3][3];  // the planes in flight, by plane mod 3
    unsigned lo[3], so[3];  // byte offsets of the lane's nodes in a plane, for loads and stores
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const bool in = (unsigned)x < (unsigned)v.nx && (unsigned)(yb + l) < (unsigned)v.ny;
        lo[l] = in ? (unsigned)(v.nx * (yb + l) + x) * (unsigned)sizeof(T) : kOff;
        so[l] = useful ? lo[l] : kOff;
#pragma unroll
        for (int k = 0; k < 3; ++k) F[k][l] = X[k][l] = R[k][l] = T(0);
    }
    const int pb = (int)(v.nxy * (long)sizeof(T));  // bytes of a plane
    const T* pf = f + v.nxy * p0;
    T* px = xo + v.nxy * (p0 - 1);
    auto load = [&](int z, T(&d)[3]) {
        const auto pl = plane(pf, pb, (unsigned)z < (unsigned)v.nz);
        pf += v.nxy;
#pragma unroll
        for (int l = 0; l < 3; ++l) bload(pl, lo[l], d[l]);
    };
#pragma unroll
    for (int k = 0; k < 3; ++k) load(p0 + k, nf[k]);
    const bool live = rows.preload(v, x, yb, p0, ze + 2 - p0, __ballot(useful));
    if (skip != 0.0) return;  // the whole grid
    if (!__syncthreads_or(live)) return;  // no unknown: x and fc are zero there already
    T acc = T(0), idn = T(0);
    auto step_as = [&](auto ph, auto fast, int p, int buf) {
        constexpr int A = decltype(ph)::value, B = (A + 2) % 3, C = (A + 1) % 3;
        constexpr bool FAST = decltype(fast)::value;
        const int i = p - p0;
        T(*wr)[W + 2][2][64] = sh[buf];
        T(*rd)[W + 2][2][64] = sh[buf ^ 1];
        T yl[3], yh[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            yl[k] = rd[k][w][1][lane];
            yh[k] = rd[k][w + 2][0][lane];
        }
#pragma unroll
        for (int l = 0; l < 3; ++l) F[A][l] = here(nf[A][l]);
        load(p + 3, nf[A]);
        // x on plane p - 1
        if (!rows.template at<FAST>(v, x, yb, p0, i - 1)) {
#pragma unroll
            for (int l = 0; l < 3; ++l) X[B][l] = T(0);
        } else {
            const int q = p - 1;
            const auto pl = plane(px, pb, q >= zs && q < ze && q < v.nz);
            T af[3];
            apply3<T>(rows.c.a, F[B], F[C], F[A], yl[0], yh[0], af);
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                const T x1 = c20 * F[B][l];
                const T d = c1 * x1 + c2 * (F[B][l] - c20 * af[l]);
                X[B][l] = x1 + d;
                bstore(pl, so[l], X[B][l]);
            }
        }
        px += v.nxy;
        // r = f - A x on plane p - 2
        if (!rows.template at<FAST>(v, x, yb, p0, i - 2)) {
#pragma unroll
            for (int l = 0; l < 3; ++l) R[C][l] = T(0);
        } else {
            T ax[3];
            apply3<T>(rows.c.a, X[C], X[A], X[B], yl[1], yh[1], ax);
#pragma unroll
            for (int l = 0; l < 3; ++l) R[C][l] = F[C][l] - ax[l];
        }
        wr[0][w + 1][0][lane] = F[A][0];
        wr[0][w + 1][1][lane] = F[A][2];
        wr[1][w + 1][0][lane] = X[B][0];
        wr[1][w + 1][1][lane] = X[B][2];
        wr[2][w + 1][0][lane] = R[C][0];
        wr[2][w + 1][1][lane] = R[C][2];
        // r - w A^T r on plane p - 3, summed over the aggregate's three planes and lines
        if (own && (FAST || i >= 6)) {
            if (rows.template at<FAST>(v, x, yb, p0, i - 3)) {
                T ar[3];
                if constexpr (SYM)
                    apply3<T>(rows.c.a, R[A], R[B], R[C], yl[2], yh[2], ar);
                else
                    apply3<T>(rows.c.at, R[A], R[B], R[C], yl[2], yh[2], ar);
#pragma unroll
                for (int l = 0; l < 3; ++l) acc += R[A][l] - omega * ar[l];
            }
            const int X_ = x / 3, Y_ = yb / 3, Z_ = (p - 3) / 3;
            const bool agg = lane >= 3 && lane < 3 + kDownX && lane % 3 == 0 && X_ < cb.mx && Y_ < cb.my;
            const long k = (X_ + 1) + cb.sx * (Y_ + 1) + cb.sxy * (Z_ + 1);
            if (A == 0 && fd && agg) idn = cb.invD[k];  // used two planes on
            if (A == 2) {
                const T s1 = shift0<false>(acc);
                const T s = acc + s1 + shift0<false>(s1);
                acc = T(0);
                if (agg) {
                    fc[k] = s;
                    if (fd) fd[k] = idn * s;
                }
            }
        }
        step_barrier();
    };
    const uint64_t steady = rows.steady(1) & ~63ull;
    auto step = [&](auto ph, int p, int buf) {
        if ((steady >> (p - p0)) & 1ull)
            step_as(ph, std::true_type{}, p, buf);
        else
            step_as(ph, std::false_type{}, p, buf);
    };
    int buf = 0;
    for (int p = p0; p < ze + 3; p += 3) {  // p0 and ze are multiples of 3
        step(std::integral_constant<int, 0>{}, p, buf);
        step(std::integral_constant<int, 1>{}, p + 1, buf ^ 1);
        step(std::integral_constant<int, 2>{}, p + 2, buf);
        buf ^= 1;
    }
}

// x' = x + P v, two Chebyshev steps on it, out = the result and partials of f . out.
template <typename T, int W>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
k_stroke_up(StrokeView<T> v, CoarseBox<T> cb,
                                                     const T* __restrict__ vc,
                                                     const T* __restrict__ xi,
                                                     const T* __restrict__ f, T* __restrict__ out,
                                                     T c1, T c2, T c20, T omega, double* part) {
    __shared__ T sh[2][2][W + 2][2][64];
    __shared__ int ring[W][3][3][64];
    __shared__ double lds[W];
    const double skip = v.skip ? *v.skip : 0.0;
    int tx, ty, sz;
    stroke_tile(v, &tx, &ty, &sz);
    const int lane = threadIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int x = kUpX * tx - 2 + lane;
    const int yb = 3 * ((W - 2) * ty + w - 1);
    const int zs = sz * v.S, ze = min(zs + v.S, v.nz);
    const int p0 = zs - 2;
    const bool own = w > 0 && w < W - 1;
    for (int i = lane + 64 * w; i < 2 * 2 * (W + 2) * 2 * 64; i += 64 * W) (&sh[0][0][0][0][0])[i] = T(0);

    Rows<T, false> rows;
    rows.ring = &ring[w][0][0][0];
    rows.init(v, yb, p0);
    T F[3][3], XP[3][3], X1[3][3];
    T nf[3][3], nx_[3][3];  // the planes in flight, by plane mod 3
    unsigned lo[3], so[3];
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const bool in = (unsigned)x < (unsigned)v.nx && (unsigned)(yb + l) < (unsigned)v.ny;
        lo[l] = in ? (unsigned)(v.nx * (yb + l) + x) * (unsigned)sizeof(T) : kOff;
        so[l] = lane >= 2 && lane < 2 + kUpX ? lo[l] : kOff;
#pragma unroll
        for (int k = 0; k < 3; ++k) F[k][l] = XP[k][l] = X1[k][l] = T(0);
    }
    const int pb = (int)(v.nxy * (long)sizeof(T));  // bytes of a plane
    const T *pf = f + v.nxy * p0, *px = xi + v.nxy * p0;
    T* po = out + v.nxy * (p0 - 2);
    auto load = [&](int z, T(&df)[3], T(&dx)[3]) {
        const bool ok = (unsigned)z < (unsigned)v.nz;
        const auto bf = plane(pf, pb, ok), bx = plane(px, pb, ok);
        pf += v.nxy;
        px += v.nxy;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            bload(bf, lo[l], df[l]);
            bload(bx, lo[l], dx[l]);
        }
    };
    // coarse values of the lane's aggregate on layers K - 1, K, K + 1, of the aggregate rows
    // before and after on layer K, and of the x-neighbour beyond the wavefront (lanes 0, 63)
    const int J = yb / 3;  // yb is a multiple of 3, at least -3
    auto col = [&](int xx, int j) {
        const int X_ = xx < 0 ? 0 : min(xx / 3, cb.mx) + 1;
        const int Y_ = min(max(j + 1, 0), cb.my + 1);
        return (unsigned)(X_ + (int)cb.sx * Y_);
    };
    const unsigned o0 = col(x, J), om = col(x, J - 1), op = col(x, J + 1),
                   oe = col(lane == 0 ? x - 1 : x + 1, J);
    auto layer = [&](int k) { return vc + cb.sxy * min(max(k + 1, 0), cb.mz + 1); };
    int K = zs / 3 - 1;  // layer of plane zs - 2
    T vm = T(0), v0 = layer(K)[o0], vp = layer(K + 1)[o0];
    T vym = layer(K)[om], vyp = layer(K)[op], ve = layer(K)[oe];
    T nvp, nym, nyp, nve;
    auto next_layer = [&]() {
        nvp = layer(K + 2)[o0];
        const T* l1 = layer(K + 1);
        nym = l1[om];
        nyp = l1[op];
        nve = l1[oe];
    };
    next_layer();
#pragma unroll
    for (int k = 0; k < 3; ++k) load(p0 + k, nf[(k + 1) % 3], nx_[(k + 1) % 3]);
    const bool live = rows.preload(v, x, yb, p0, ze + 2 - p0,
                                   __ballot(own && lane >= 2 && lane < 2 + kUpX));
    if (skip != 0.0) return;
    if (!__syncthreads_or(live)) {
        if (part && lane == 0 && w == 0) part[blockIdx.x] = 0.0;
        return;
    }
    double dsum = 0.0;
    // zeros where the node of plane z is not an unknown
    auto mask_z = [&](int z, T(&e)[3]) {
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            uint64_t u = 0;
            if ((unsigned)z < (unsigned)v.nz && lo[l] != kOff)
                u = v.unk[((long)z * v.ny + yb + l) * v.nsegx + (x >> 6)] >> (x & 63);
            e[l] = u & 1ull ? e[l] : T(0);
        }
        settle(e);
    };
    auto step_as = [&](auto ph, auto fast, int p, int buf) {
        constexpr int A = decltype(ph)::value, B = (A + 2) % 3, C = (A + 1) % 3;
        constexpr bool FAST = decltype(fast)::value;
        const int i = p - p0;
        T(*wr)[W + 2][2][64] = sh[buf];
        T(*rd)[W + 2][2][64] = sh[buf ^ 1];
        T yl[2], yh[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            yl[k] = rd[k][w][1][lane];
            yh[k] = rd[k][w + 2][0][lane];
        }
        T xin[3];
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            F[A][l] = here(nf[A][l]);
            xin[l] = here(nx_[A][l]);
        }
        if (A == 0) {  // the next layer of aggregates
            ++K;
            vm = v0;
            v0 = vp;
            vp = nvp;
            vym = nym;
            vyp = nyp;
            ve = nve;
            next_layer();
        }
        load(p + 3, nf[A], nx_[A]);
        if (!rows.template at<FAST>(v, x, yb, p0, i)) {
#pragma unroll
            for (int l = 0; l < 3; ++l) XP[A][l] = T(0);
        } else {
            const T xm = wave_shift<true>(v0, ve), xp = wave_shift<false>(v0, ve);
            T zm[3], zp[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                zm[l] = A == 0 ? vm : v0;
                zp[l] = A == 2 ? vp : v0;
            }
            // P v is zero off the unknowns.  Rows hold zeros towards neighbours in x and y that
            // are none, but along z they may stand for several planes: where the line changes
            // from plane to plane its neighbours are masked
            if (!FAST && ((rows.change >> i) & 3ull)) {
                mask_z(p - 1, zm);
                mask_z(p + 1, zp);
            }
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                const T ym = l ? v0 : vym, yp = l < 2 ? v0 : vyp;
                const T(&a)[6] = rows.c.a[l];
                const T ae = v0 + a[0] * xm + a[1] * xp + a[2] * ym + a[3] * yp + a[4] * zm[l] +
                             a[5] * zp[l];
                const T o = xin[l] + (v0 - omega * ae);
                XP[A][l] = (rows.c.um[l] >> lane) & 1ull ? o : T(0);
            }
        }
        if (!rows.template at<FAST>(v, x, yb, p0, i - 1)) {
#pragma unroll
            for (int l = 0; l < 3; ++l) X1[B][l] = T(0);
        } else {
            T ax[3];
            apply3<T>(rows.c.a, XP[B], XP[C], XP[A], yl[0], yh[0], ax);
#pragma unroll
            for (int l = 0; l < 3; ++l) X1[B][l] = XP[B][l] + c20 * (F[B][l] - ax[l]);
        }
        wr[0][w + 1][0][lane] = XP[A][0];
        wr[0][w + 1][1][lane] = XP[A][2];
        wr[1][w + 1][0][lane] = X1[B][0];
        wr[1][w + 1][1][lane] = X1[B][2];
        if (own && (FAST || i >= 4) && rows.template at<FAST>(v, x, yb, p0, i - 2)) {
            T ax[3];
            apply3<T>(rows.c.a, X1[C], X1[A], X1[B], yl[1], yh[1], ax);
            const auto pl = plane(po, pb, true);
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                const T d = c1 * (X1[C][l] - XP[C][l]) + c2 * (F[C][l] - ax[l]);
                const T z = X1[C][l] + d;
                bstore(pl, so[l], z);
                dsum += so[l] != kOff ? (double)F[C][l] * (double)z : 0.0;
            }
        }
        po += v.nxy;
        step_barrier();
    };
    const uint64_t steady = rows.steady(0) & ~(rows.change >> 1) & ~15ull;
    auto step = [&](auto ph, int p, int buf) {
        if ((steady >> (p - p0)) & 1ull)
            step_as(ph, std::true_type{}, p, buf);
        else
            step_as(ph, std::false_type{}, p, buf);
    };
    int buf = 0;
    for (int p = p0; p < ze + 2; p += 3) {  // p0 = 1 mod 3
        step(std::integral_constant<int, 1>{}, p, buf);
        if (p + 1 < ze + 2) step(std::integral_constant<int, 2>{}, p + 1, buf ^ 1);
        if (p + 2 < ze + 2) step(std::integral_constant<int, 0>{}, p + 2, buf);
        buf ^= 1;
    }
    const double s = block_sum(dsum, lds);
    if (part && lane == 0 && w == 0) part[blockIdx.x] = s;
}

// ---- what the strokes know of each line
//
// The rows of a line (y, z) may stand for those of the line one plane below when both have
// the same unknowns and, at every unknown, rows that agree in each coefficient whose
// neighbour is an unknown of both lines' surroundings: along z the end planes of a pipe
// lack a neighbour, whose coefficient is free because the value there is zero.  A pipe of
// constant cross-section is then one group from end to end.  The rows of a group are read
// from one of its planes that has both z-neighbours: the plane itself, the one above the
// group's first, or the one below its last.  A group of two planes has none and is split.

// One wavefront per line: compat[y][z] = 1 where the rows of (y, z - 1) may stand for
// (y, z)'s, and 2 where the line has an unknown.
__global__ void __launch_bounds__(kThreads) k_zcompat(L0View<double> v, uint8_t* __restrict__ compat) {
    const long line = (long)blockIdx.x * kBlockY + threadIdx.y;
    if (line >= (long)v.ny * v.nz) return;
    const int lane = threadIdx.x, z = (int)(line / v.ny), y = (int)(line % v.ny);
    const long step = (long)v.ny * v.nsegx;
    bool ok = true, any = false;
    for (int q = 0; q < v.nsegx; ++q) {
        const long s1 = line * v.nsegx + q, s0 = s1 - step;
        const uint64_t u = v.unk[s1];
        any = any || u != 0;
        if (z == 0) {
            ok = ok && u == 0;
            continue;
        }
        if (u != v.unk[s0]) {
            ok = false;
            continue;
        }
        const uint64_t r1 = v.irr[s1], r0 = v.irr[s0];
        if (u == 0 || (r1 == r0 && (r1 == 0 || v.base[s1] == v.base[s0]))) continue;
        // whether the z-neighbours beyond the pair are unknowns
        const bool below = z >= 2 && ((v.unk[s0 - step] >> lane) & 1ull);
        const bool above = z + 1 < v.nz && ((v.unk[s1 + step] >> lane) & 1ull);
        bool same = true;
        if ((u >> lane) & 1ull) {
            const uint64_t m = (1ull << lane) - 1ull;
            const bool i1 = (r1 >> lane) & 1ull, i0 = (r0 >> lane) & 1ull;
            const long k1 = v.base[s1] + (int)__popcll(r1 & m), k0 = v.base[s0] + (int)__popcll(r0 & m);
            for (int d = 0; d < 6; ++d) {
                if ((d == 4 && !below) || (d == 5 && !above)) continue;
                const double c = v.c[d >> 1];
                const double a1 = i1 ? v.tcoef(d, k1) : c, a0 = i0 ? v.tcoef(d, k0) : c;
                const double t1 = i1 ? v.tcoefT(d, k1) : c, t0 = i0 ? v.tcoefT(d, k0) : c;
                same = same && a1 == a0 && t1 == t0;
            }
        }
        if (__ballot(!same) != 0) ok = false;
    }
    if (lane == 0) compat[(long)v.nz * y + z] = (ok ? 1 : 0) | (any ? 2 : 0);
}

// zinfo[y][z], z = 0..nz: kZSame where the line's rows are those of the line below, kZUnk
// where it has an unknown, and from bit kZRep 1 + (the plane its rows are read from - z).
__global__ void __launch_bounds__(256) k_zinfo(int ny, int nz, const uint8_t* __restrict__ compat,
                                               uint8_t* __restrict__ zinfo) {
    const long t = blockIdx.x * 256L + threadIdx.x;
    if (t >= (long)ny * (nz + 1)) return;
    const int y = (int)(t / (nz + 1)), z = (int)(t % (nz + 1));
    const uint8_t* c = compat + (long)nz * y;
    if (z == nz) {  // above the box: as an empty line
        zinfo[t] = ((c[nz - 1] & 2) ? 0 : kZSame) | (1 << kZRep);
        return;
    }
    auto same = [&](int k) { return k >= 0 && k < nz && (c[k] & 1); };  // plane k continues a group
    bool s = same(z);
    int rep = 0;
    if (s && !same(z - 1) && !same(z + 1)) {
        s = false;  // the second of two planes
    } else if (s && !same(z + 1)) {
        rep = -1;  // the last of at least three
    } else if (!s && same(z + 1) && same(z + 2)) {
        rep = 1;  // the first of at least three
    }
    zinfo[t] = (s ? kZSame : 0) | ((c[z] & 2) ? kZUnk : 0) | ((1 + rep) << kZRep);
}

// out[2 Y], out[2 Y + 1]: the planes where aggregate row Y's rows change, beyond its first, and its
// planes with unknowns.
__global__ void __launch_bounds__(64) k_zchange(int ny, int nz, const uint8_t* __restrict__ zinfo,
                                                int* __restrict__ out) {
    const int y0 = 3 * blockIdx.x;
    int change = 0, planes = 0;
    for (int z = threadIdx.x; z < nz; z += kWave) {
        int all = kZSame, any = 0;
        for (int y = y0; y < min(y0 + 3, ny); ++y) {
            const int v = zinfo[(long)(nz + 1) * y + z];
            all &= v;
            any |= v;
        }
        planes += (any & kZUnk) != 0;
        change += (any & kZUnk) != 0 && !(all & kZSame);
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        change += __shfl_xor(change, o);
        planes += __shfl_xor(planes, o);
    }
    if (threadIdx.x != 0) return;
    out[2 * blockIdx.x] = max(change - 1, 0);
    out[2 * blockIdx.x + 1] = planes;
}

long zinfo_bytes(const FineLevel& L) { return (long)L.ny * (L.nz + 1); }

static StrokeTile stroke_tiling(const FineLevel& L, const std::vector<uint64_t>& shadow, bool up,
                                int bytes, std::vector<TileAt>* tiles);
static std::vector<TileAt> live_tiles(const FineLevel& L, const std::vector<uint64_t>& shadow,
                                       int tx, int lines);

// Which nodes of the (x, y) cross-section hold an unknown on any plane: OR of the unknown
// masks over z, 32 planes a thread.
__global__ void __launch_bounds__(256) k_shadow(int nz, long words, const uint64_t* __restrict__ unk,
                                                uint64_t* __restrict__ shadow) {
    const long t = blockIdx.x * 256L + threadIdx.x;
    if (t >= words) return;
    uint64_t m = 0;
    const int z1 = min(nz, 32 * (int)(blockIdx.y + 1));
    for (int z = 32 * blockIdx.y; z < z1; ++z) m |= unk[words * z + t];
    if (m) atomicOr((unsigned long long*)&shadow[t], (unsigned long long)m);
}

void l0_zinfo(FineLevel& L, bool counts, hipStream_t s) {
    if (!L.zinfo) L.zinfo = (uint8_t*)dmalloc(zinfo_bytes(L), false);
    // the unknowns never change, and with them neither do the tiles: the first time only
    const bool first = L.stroke[0][0].W == 0;
    const long lines = (long)L.ny * L.nz, nrow = counts ? (L.ny + 2) / 3 : 0,
               words = first ? (long)L.ny * L.nsegx : 0;
    // the shadow, two counts an aggregate row, and a byte a line
    Tmp sh(8 * (words + nrow) + lines, false);
    uint8_t* compat = (uint8_t*)(sh.as<uint64_t>() + words + nrow);
    hipLaunchKernelGGL(k_zcompat, dim3((unsigned)((lines + kBlockY - 1) / kBlockY)),
                       dim3(kWave, kBlockY), 0, s, L.view<double>(), compat);
    hipLaunchKernelGGL(k_zinfo, dim3((unsigned)((zinfo_bytes(L) + 255) / 256)), dim3(256), 0, s,
                       L.ny, L.nz, (const uint8_t*)compat, L.zinfo);
    std::vector<uint64_t> got(words + nrow);
    if (counts)
        hipLaunchKernelGGL(k_zchange, dim3((unsigned)nrow), dim3(kWave), 0, s, L.ny, L.nz,
                           (const uint8_t*)L.zinfo, (int*)(sh.as<uint64_t>() + words));
    if (first) {
        zero_fill(sh.p, 8 * words, s);
        hipLaunchKernelGGL(k_shadow, dim3((unsigned)((words + 255) / 256), (unsigned)((L.nz + 31) / 32)),
                           dim3(256), 0, s, L.nz, words, (const uint64_t*)L.unk, sh.as<uint64_t>());
    }
    HIPCHECK(hipGetLastError());
    if (!got.empty())
        HIPCHECK(hipMemcpyAsync(got.data(), sh.p, 8 * got.size(), hipMemcpyDeviceToHost, s));
    HIPCHECK(hipStreamSynchronize(s));  // also: the temporary may go
    long change = 0, planes = 0;
    L.change_worst = 0.0;
    for (long Y = 0; Y < nrow; ++Y) {
        int n[2];
        std::memcpy(n, &got[words + Y], 8);
        change += n[0];
        planes += n[1];
        if (n[1]) L.change_worst = std::max(L.change_worst, (double)n[0] / n[1]);
    }
    L.change_mean = planes ? (double)change / planes : 0.0;
    if (!first) return;
    const std::vector<uint64_t>& shadow = got;
    std::vector<TileAt> lists;
    for (int d = 0; d < 2; ++d)
        for (int up = 0; up < 2; ++up) {
            std::vector<TileAt> tiles;
            StrokeTile& t = L.stroke[d][up];
            t = stroke_tiling(L, shadow, up != 0, d ? 8 : 4, &tiles);
            t.list = (int)lists.size();
            lists.insert(lists.end(), tiles.begin(), tiles.end());
        }
    {
        const std::vector<TileAt> tiles = live_tiles(L, shadow, kColX, kColLines);
        L.col.live = (int)tiles.size();
        L.col.list = (int)lists.size();
        // 12 planes a slab, 6 where that leaves compute units with less than two blocks (128 x 128
        // x 256 fp64: 57 us with 6, 59 with 12, 63 with 3; 145 x 145 x 435: 156, 146, 180)
        for (L.col.S = 12; ; L.col.S = 6) {
            L.col.gz = (L.nz + L.col.S - 1) / L.col.S;
            if (L.col.S == 6 || L.col.blocks() >= 512) break;
        }
        lists.insert(lists.end(), tiles.begin(), tiles.end());
    }
    L.n_tiles = (long)lists.size();
    const size_t bytes = sizeof(TileAt) * lists.size();
    L.tiles = (TileAt*)dmalloc(bytes, false);
    HIPCHECK(hipMemcpyAsync(L.tiles, lists.data(), bytes, hipMemcpyHostToDevice, s));
    HIPCHECK(hipStreamSynchronize(s));  // the host list goes
}

// The tiles of the cross-section that hold an unknown.
static std::vector<TileAt> live_tiles(const FineLevel& L, const std::vector<uint64_t>& shadow,
                                       int tx, int lines) {
    std::vector<TileAt> out;
    for (int j = 0; j * lines < L.ny; ++j)
        for (int i = 0; i * tx < L.nx; ++i) {
            const int x0 = i * tx, x1 = std::min(L.nx, x0 + tx), y1 = std::min(L.ny, lines * (j + 1));
            bool any = false;
            for (int y = lines * j; y < y1 && !any; ++y)
                for (int q = x0 >> 6; q <= (x1 - 1) >> 6 && !any; ++q) {
                    uint64_t m = shadow[(long)y * L.nsegx + q];
                    if (x0 > 64 * q) m &= ~0ull << (x0 - 64 * q);
                    if (x1 < 64 * q + 64) m &= ~0ull >> (64 * q + 64 - x1);
                    any = m != 0;
                }
            if (any) out.push_back({i, j});
        }
    return out;
}

// Tile of a stroke: wavefronts per block and planes per slab.  More wavefronts re-read and
// recompute fewer halo lines (3 W - 6 of 3 W are outputs) and longer slabs fewer halo planes,
// while a launch whose last round of blocks is nearly empty, or that leaves compute units
// without work, loses more than the halo: the choice minimises a model of the time,
//   start + (S + halo) sum over rounds of (a + b n),
// with n wavefronts per SIMD and the blocks that hold unknowns.  a and b are the microseconds
// of a plane step measured on boxes from 33^3 to 256 x 256 x 768 (fp32, 8 wavefronts a block:
// 0.79 us with one block on a compute unit, 1.18 with two; fp64: 0.50 with one wavefront per
// SIMD, 0.87 with two).  Single launches (down / up): 128 x 128 x 256 ellipse in fp64, 8 wavefronts,
// 24 planes 30.5 / 35.7 us, 27 planes 32.6 / 38.5, 21 planes (a second round begun) 49.7 / 60.1, 12
// planes 38.8 / 45.9; 256 x 256 x 768 ellipse in fp32, 16 wavefronts, 48 planes 145 / 179 us, 54 planes
// 141 / 198, 24 planes 150 / 189, 57 planes 166 / 203.
static StrokeTile stroke_tiling(const FineLevel& L, const std::vector<uint64_t>& shadow, bool up,
                                int bytes, std::vector<TileAt>* tiles) {
    const int tx = up ? kUpX : kDownX;
    StrokeTile best;
    double t_best = 0.0;
    for (int W : {4, 8, 16}) {
        if (bytes == 8 && W == 16) break;  // fp64: 128 registers a lane do not hold the state
        const int per_cu = (bytes == 4 ? 16 : 8) / W;  // blocks that fit a compute unit's registers
        const double a = bytes == 4 ? 0.38 : 0.15, b = bytes == 4 ? 0.20 : 0.36;
        const std::vector<TileAt> list = live_tiles(L, shadow, tx, 3 * (W - 2));
        StrokeTile t;
        t.W = W;
        t.live = (int)list.size();
        bool better = false;
        for (t.S = 3; t.S <= kStrokeMaxPlanes; t.S += 3) {
            t.gz = (L.nz + t.S - 1) / t.S;
            const long slots = 256L * per_cu, full = t.blocks() / slots, rest = t.blocks() % slots;
            const double n1 = (double)W / 4;  // wavefronts per SIMD of one block
            double round = full * (a + b * n1 * per_cu);
            if (rest) round += a + b * n1 * ((rest + 255) / 256);
            const double us = 4.0 + (t.S + 6) * round;
            if (best.W == 0 || us < t_best) {
                best = t;
                t_best = us;
                better = true;
            }
        }
        if (better) *tiles = list;
    }
    return best;
}

template <typename T>
static StrokeView<T> stroke_view(const FineLevel& L, const StrokeTile& t) {
    const L0View<T> l = L.view<T>();
    StrokeView<T> v;
    v.nx = L.nx; v.ny = L.ny; v.nz = L.nz; v.nsegx = L.nsegx; v.nxy = L.nxy;
    v.unk = l.unk; v.irr = l.irr; v.base = l.base; v.tab = l.tab; v.tabT = l.tabT;
    for (int a = 0; a < 3; ++a) v.c[a] = l.c[a];
    v.zinfo = L.zinfo;
    v.tiles = L.tiles + t.list;
    v.live = t.live;
    v.S = t.S;
    v.skip = l.skip;
    return v;
}

template <typename T>
static CoarseBox<T> coarse_box(const CoarseLevel& C) {
    CoarseBox<T> b;
    b.mx = C.mx; b.my = C.my; b.mz = C.mz;
    b.sx = C.sx; b.sxy = C.sxy;
    b.invD = sizeof(T) == 8 ? (const T*)C.invD64 : (const T*)C.invD32;
    return b;
}

// Strokes need the degree-2 smoother and planes that a 32-bit byte offset reaches, and pay where
// lines keep their rows from plane to plane: a plane where a line changes reads rows in each
// stage, two dependent trips to memory behind one another, and so do the planes after it.  The line
// lies where the two forms met, in the share of changing planes (solves of 8 steps, by steps /
// by strokes, of pipes whose radius changes every few planes, pipes with open ends, cavities with
// bores, tapers, spheres and pipes along x and y, from 24^3 to 256^3):
//   below 800 thousand nodes a launch lasts as long as its slowest block, and one change inside a
//   slab costs what strokes save: 64 x 64 x 128 closed 1.17, with open ends (share 0.03) 1.05,
//   49 x 49 x 98 with open ends (0.04) 1.02, 40^3 (0.10) 0.98, 33^3 cavity (0.32) 0.85, sphere
//   0.76, 64 x 64 x 128 cavity (0.08) 0.88, which keeps strokes' fewer launches for batches;
//   up to 3 million 96 x 96 x 192 with a share of 0.43 1.0, 0.27 1.1, each plane 0.76;
//   above 128 x 128 x 256 0.71: 1.06, each plane 0.93;
//   rows longer than 128 nodes that miss the 16-byte lanes are slow by steps: with a change on
//   each plane 139^3 1.2 in fp64 and 1.0 in fp32, 131 x 131 x 262 and 161 x 161 x 322 1.1 to 1.2,
//   above 10 million 199 x 199 x 300 0.95 and 1.0;
//   with 16-byte lanes 256^3 fp64 0.29: 1.0, fp32 0.45: 1.0, each plane 0.66 and 0.83.
// On one-node lanes a change anywhere holds up the launch, so the worst aggregate row counts
// as much as the mean (pipes along x, whose lines beside the wall change on every plane).
bool l0_strokes(const FineLevel& L, int degree, int bytes) {
    if (degree != 2 || L.nxy * bytes >= (long)kOff) return false;
    double most;
    if (L.nbox < 800000)
        most = 0.1;
    else if (L.wide)
        most = bytes == 8 ? 0.3 : 0.45;
    else if (L.nx > 128 && L.nbox <= 10000000)
        most = bytes == 8 || L.nbox >= 3000000 ? 1.0 : 0.75;
    else
        most = L.nbox < 3000000 ? 0.4 : 0.75;
    return l0_change(L) <= most;
}

double l0_change(const FineLevel& L) {
    return L.wide ? L.change_mean : 0.5 * (L.change_mean + L.change_worst);
}

long l0_stroke_parts(const FineLevel& L, int bytes) { return L.stroke[bytes == 8][1].blocks(); }

// Bytes of a stroke: level-0 vectors it reads or writes, the coarse vector, and per line the
// z-information (masks and table rows only where a line changes along z).
static long stroke_bytes(const FineLevel& L, const CoarseLevel& C, int vecs, int coarse, long w) {
    return (vecs * L.n_unknowns + coarse * C.n_unknowns) * w + zinfo_bytes(L);
}

template <typename T>
void l0_down(const FineLevel& L, const CoarseLevel& C, bool sym, const T* f, T* x, T* fc, T* fd,
             double c1, double c2, double c20, double omega, hipStream_t s) {
    const StrokeTile& t = L.stroke[sizeof(T) == 8][0];
    const StrokeView<T> v = stroke_view<T>(L, t);
    const CoarseBox<T> cb = coarse_box<T>(C);
    const dim3 g((unsigned)t.blocks()), b(kWave, t.W);
    const long by = stroke_bytes(L, C, 2, fd ? 3 : 1, sizeof(T));
    KTimer kt(s, {{T_L0_CHEB, by / 3}, {T_L0_RESID, by / 3}, {T_L0_RESTRICT, by / 3}});
#define DOWN(W_, SYM_)                                                                         \
    klaunch(kt, true, (k_stroke_down<T, SYM_, W_>), g, b, v, cb, f, x, fc, fd, (T)c1, (T)c2,    \
            (T)c20, (T)omega)
    if (t.W == 4 && sym) DOWN(4, true);
    else if (t.W == 4) DOWN(4, false);
    else if (t.W == 8 && sym) DOWN(8, true);
    else if (t.W == 8) DOWN(8, false);
    else if constexpr (sizeof(T) == 4) {
        if (sym) DOWN(16, true);
        else DOWN(16, false);
    }
#undef DOWN
    HIPCHECK(hipGetLastError());
}
template void l0_down<double>(const FineLevel&, const CoarseLevel&, bool, const double*, double*,
                              double*, double*, double, double, double, double, hipStream_t);
template void l0_down<float>(const FineLevel&, const CoarseLevel&, bool, const float*, float*,
                             float*, float*, double, double, double, double, hipStream_t);

template <typename T>
void l0_up(const FineLevel& L, const CoarseLevel& C, const T* vc, const T* x, const T* f, T* out,
           double c1, double c2, double c20, double omega, double* dot, hipStream_t s) {
    const StrokeTile& t = L.stroke[sizeof(T) == 8][1];
    const StrokeView<T> v = stroke_view<T>(L, t);
    const CoarseBox<T> cb = coarse_box<T>(C);
    const dim3 g((unsigned)t.blocks()), b(kWave, t.W);
    const long by = stroke_bytes(L, C, 3, 1, sizeof(T));
    KTimer kt(s, {{T_L0_PROLONG, by / 3}, {T_L0_CHEB, by / 3 * 2}});
#define UP(W_)                                                                                 \
    klaunch(kt, true, (k_stroke_up<T, W_>), g, b, v, cb, vc, x, f, out, (T)c1, (T)c2, (T)c20,   \
            (T)omega, dot)
    if (t.W == 4) UP(4);
    else if (t.W == 8) UP(8);
    else if constexpr (sizeof(T) == 4) UP(16);
#undef UP
    HIPCHECK(hipGetLastError());
}
template void l0_up<double>(const FineLevel&, const CoarseLevel&, const double*, const double*,
                            const double*, double*, double, double, double, double, double*,
                            hipStream_t);
template void l0_up<float>(const FineLevel&, const CoarseLevel&, const float*, const float*,
                           const float*, float*, double, double, double, double, double*,
                           hipStream_t);

}  // namespace saamg
