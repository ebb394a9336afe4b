// Particle coupling on either side of the solve (Section 1 and Section 4): cloud-in-cell
// deposition of particle charge to the lattice, and the field E = -grad(phi) interpolated
// back to the particles with the same trilinear weights.
//
// Deposition is deterministic in fp64 without floating-point atomics: particles are keyed by
// lattice cell and stably sorted; chunks of kChunk sorted particles sum the eight corner
// weights of each run of equal cells they hold, and each node sums the runs of its (up to)
// eight adjacent cells in a fixed order.  The work follows the particles, not the cells, so a
// bunch that puts thousands of particles into one cell costs what a spread one does (one
// thread a node that read its cells' particles one by one took 535 us of a 49x49x97 step
// with 100 thousand particles, 150 in the fullest cell; the run sums and the node pass take 8
// and 21 us; 192x192x1024 with 2 million: 684 us and 90 of clears before, 55 and 161 now).
// The gather differences phi centrally at the eight corner nodes of each particle's cell.
#include <hipcub/hipcub.hpp>

#include "launch.h"

namespace saamg {

struct PicView {
    int nx, ny, nz, zoff;    // box, and the box plane of the lattice's plane 0
    int nxl, nyl, nzl;       // lattice nodes
    double ox, oy, oz;       // lattice node (0, 0, 0)
    double hx, hy, hz;
    double rob;              // 2 h_z / d for open ends, else 0
};

// Lattice cell of a position and the fractional offsets in it; false if outside.
__device__ inline bool pic_cell(const PicView& v, double px, double py, double pz, int* ci,
                                int* cj, int* ck, double* fx, double* fy, double* fz) {
    const double ux = (px - v.ox) / v.hx, uy = (py - v.oy) / v.hy, uz = (pz - v.oz) / v.hz;
    const double gx = floor(ux), gy = floor(uy), gz = floor(uz);
    // reject before converting, so that far-away particles cannot overflow the cast
    if (!(gx >= 0.0 && gx <= v.nxl - 2 && gy >= 0.0 && gy <= v.nyl - 2 && gz >= 0.0 &&
          gz <= v.nzl - 2))
        return false;
    *ci = (int)gx;
    *cj = (int)gy;
    *ck = (int)gz;
    *fx = ux - gx;
    *fy = uy - gy;
    *fz = uz - gz;
    return true;
}

__global__ void k_pic_keys(PicView v, const double* __restrict__ pos, long n, uint32_t sentinel,
                           uint32_t* __restrict__ key, int32_t* __restrict__ idx) {
    const long p = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (p >= n) return;
    int i, j, k;
    double fx, fy, fz;
    const bool in = pic_cell(v, pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], &i, &j, &k, &fx, &fy, &fz);
    key[p] = in ? (uint32_t)(i + (long)(v.nxl - 1) * (j + (long)(v.nyl - 1) * k)) : sentinel;
    idx[p] = (int32_t)p;
}

// Sorted particles per chunk: one block of the run sums.
constexpr int kChunk = 256;

// First position in [lo, hi) of the sorted keys whose key is not below v.
__device__ inline int pic_lower(const uint32_t* __restrict__ key, int lo, int hi, uint32_t v) {
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (key[mid] < v)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Blocks below nchunk: the corner sums of each run of equal cells in chunk b.  The sum of a
// run that begins here goes to `run` at the slot of its cell (`by_cell`) or of its first
// particle, that of a run continued from the chunk before to `carry` at the chunk.
// Eight threads sum a run, one per corner, so the longest chain is kChunk additions and the
// stores are 64-byte lines.  `cell` receives where an occupied cell's run begins; the entries
// of empty cells are left as they are (any value: k_pic_nodes checks an entry against the
// key it points to), so the array is not cleared.  Blocks from nchunk on: where each lattice
// row of cells begins among the sorted particles (row nrow: where the particles inside end);
// with it the nodes of empty rows look at no cell.  A start and an end per cell, cleared and
// read at every node, were 300 MB on a 192 x 192 x 1024 lattice.
__global__ __launch_bounds__(kChunk) void k_pic_runs(PicView v, const double* __restrict__ pos,
                                                     const uint32_t* __restrict__ key,
                                                     const int32_t* __restrict__ idx, int n, int nchunk,
                                                     uint32_t sentinel, double q, bool by_cell, long nrow,
                                                     double* __restrict__ run, double* __restrict__ carry,
                                                     int32_t* __restrict__ cell, int32_t* __restrict__ row) {
    __shared__ double w[8][kChunk];
    __shared__ uint32_t ks[kChunk];
    __shared__ int start[kChunk + 1];
    __shared__ int count[kChunk / 64];
    const int t = threadIdx.x;
    if ((int)blockIdx.x >= nchunk) {
        const long r = ((long)blockIdx.x - nchunk) * kChunk + t;
        if (r <= nrow) row[r] = pic_lower(key, 0, n, (uint32_t)(r * (v.nxl - 1)));
        return;
    }
    const long s = (long)blockIdx.x * kChunk + t;
    const uint32_t k = s < n ? key[s] : sentinel;
    const uint32_t before = s > 0 && s < n ? key[s - 1] : sentinel;
    ks[t] = k;
    const bool head = t == 0 || (s < n && k != before);
    const unsigned long long heads = __ballot(head);
    if ((t & 63) == 0) count[t >> 6] = __popcll(heads);
    if (k != sentinel) {
        const long p = idx[s];
        int a, b, e;
        double fx, fy, fz;
        pic_cell(v, pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], &a, &b, &e, &fx, &fy, &fz);
        for (int c = 0; c < 8; ++c)
            w[c][t] = q * ((c & 1) ? fx : 1.0 - fx) * ((c & 2) ? fy : 1.0 - fy) * ((c & 4) ? fz : 1.0 - fz);
    }
    __syncthreads();
    int at = 0, nrun = 0;
    for (int g = 0; g < kChunk / 64; ++g) {
        if (g < (t >> 6)) at += count[g];
        nrun += count[g];
    }
    at += __popcll(heads & ((1ull << (t & 63)) - 1));
    if (head) start[at] = t;
    if (t == 0) start[nrun] = (int)min((long)kChunk, n - (long)blockIdx.x * kChunk);
    __syncthreads();
    for (int p = t; p < 8 * nrun; p += kChunk) {
        const int r = p >> 3, c = p & 7, b = start[r], e = start[r + 1];
        const uint32_t kr = ks[b];
        if (kr == sentinel) continue;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        int i = b;
        for (; i + 3 < e; i += 4) {
            a0 += w[c][i];
            a1 += w[c][i + 1];
            a2 += w[c][i + 2];
            a3 += w[c][i + 3];
        }
        for (; i < e; ++i) a0 += w[c][i];
        const double sum = (a0 + a1) + (a2 + a3);
        const long first = (long)blockIdx.x * kChunk + b;
        if (b == 0 && first > 0 && key[first - 1] == kr) {
            carry[8 * (long)blockIdx.x + c] = sum;
        } else {
            run[8 * (by_cell ? (long)kr : first) + c] = sum;
            if (c == 0) cell[kr] = (int32_t)first;
        }
    }
}

// Adds corners c and c + 4 (z = 0 and 1) of the cell whose sorted particles begin at b: the
// run that begins there and its continuations, one per chunk that it reaches into.
__device__ inline void pic_corners(const uint32_t* __restrict__ key, const double* __restrict__ run,
                                   const double* __restrict__ carry, bool by_cell, uint32_t cell, int b,
                                   int hi, int c, double& dn, double& up) {
    const double* r = run + 8 * (by_cell ? (long)cell : (long)b) + c;
    double d = r[0], u = r[4];
    for (int g = b / kChunk + 1; (long)g * kChunk < hi && key[(long)g * kChunk] == cell; ++g) {
        d += carry[8 * (long)g + c];
        u += carry[8 * (long)g + c + 4];
    }
    dn += d;
    up += u;
}

// Box nodes: kPicPlanes consecutive planes per thread, so that the row starts of a column
// are loaded together and a node of an empty neighbourhood costs its store (most of the box:
// a bunch fills a few percent of it).  Bound by that store, 8 bytes a node.
constexpr int kPicPlanes = 4;
__global__ __launch_bounds__(256) void k_pic_nodes(PicView v, const uint32_t* __restrict__ key,
                                                   const int32_t* __restrict__ row,
                                                   const int32_t* __restrict__ cell,
                                                   const double* __restrict__ run,
                                                   const double* __restrict__ carry, bool by_cell,
                                                   double* __restrict__ rho) {
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x, nxy = (long)v.nx * v.ny;
    if (t >= nxy) return;
    int i, j;
    if (nxy <= 0xffffffffl) {
        j = (int)((uint32_t)t / (uint32_t)v.nx);
        i = (int)((uint32_t)t - (uint32_t)j * (uint32_t)v.nx);
    } else {
        j = (int)(t / v.nx);
        i = (int)(t - (long)j * v.nx);
    }
    const double vol = v.hx * v.hy * v.hz;
    for (long kb = (long)blockIdx.y * kPicPlanes; kb < v.nz; kb += (long)gridDim.y * kPicPlanes) {
        // the sorted particles of cell rows (j - 1 + y, k - 1 + z): [lo, hi)
        int lo[kPicPlanes + 1][2], hi[kPicPlanes + 1][2];
#pragma unroll
        for (int z = 0; z <= kPicPlanes; ++z) {
            const long cz = kb - v.zoff - 1 + z;
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int cy = j - 1 + y;
                const bool in = cz >= 0 && cz <= v.nzl - 2 && cy >= 0 && cy <= v.nyl - 2;
                const long r = in ? cy + (long)(v.nyl - 1) * cz : 0;
                const int a = row[r], b = row[r + 1];
                lo[z][y] = a;
                hi[z][y] = in ? b : a;
            }
        }
        // cells (i - 1, i) of each row, once for the two node planes it belongs to
        double low[2] = {0.0, 0.0};  // sums of the row plane below, as its upper corners
#pragma unroll
        for (int z = 0; z <= kPicPlanes; ++z) {
            double up[2] = {0.0, 0.0}, dn[2] = {0.0, 0.0};
            if (lo[z][0] < hi[z][0] || lo[z][1] < hi[z][1]) {
                int at[2][2];
                uint32_t base[2];
                bool has[2][2];
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    base[y] = (uint32_t)((v.nxl - 1) * (j - 1 + y + (v.nyl - 1) * (kb - v.zoff - 1 + z)) + i);
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        has[y][x] = lo[z][y] < hi[z][y] && i - 1 + x >= 0 && i - 1 + x <= v.nxl - 2;
                        at[y][x] = has[y][x] ? cell[base[y] - 1 + x] : 0;
                    }
                }
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        has[y][x] = has[y][x] && at[y][x] >= lo[z][y] && at[y][x] < hi[z][y] &&
                                    key[at[y][x]] == base[y] - 1 + x;
                // the node is corner x = 1 of cell i - 1 and x = 0 of cell i; y = 1 of row j - 1
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        if (has[y][x])
                            pic_corners(key, run, carry, by_cell, base[y] - 1 + x, at[y][x], hi[z][y],
                                        (1 - x) + 2 * (1 - y), dn[y], up[y]);
            }
            // dn: node plane k = this row plane (z = 0 corners); low: the plane below's z = 1
            const long kn = kb - 1 + z;  // box plane whose two row planes are now both known
            if (z > 0 && kn < v.nz) rho[t + nxy * kn] = ((low[0] + low[1]) + (dn[0] + dn[1])) / vol;
            low[0] = up[0];
            low[1] = up[1];
        }
    }
}

// phi at box node (i, j, kb) as the field differences see it: 0 off the domain and beyond
// the box; beyond an open end (the ghost planes) eq. inlet's u(x'') - (2 h_z / d) u(x).
__device__ inline double pic_phi(const PicView& v, const double* __restrict__ phi,
                                 const uint8_t* __restrict__ mask, int i, int j, int kb) {
    if (i < 0 || j < 0 || i >= v.nx || j >= v.ny) return 0.0;
    if (v.rob > 0.0 && (kb == 0 || kb == v.nz - 1)) {
        const int ke = kb == 0 ? 1 : v.nz - 2, ki = kb == 0 ? 2 : v.nz - 3;
        const long e = i + (long)v.nx * (j + (long)v.ny * ke);
        if (!mask[e]) return 0.0;
        const long in = i + (long)v.nx * (j + (long)v.ny * ki);
        return (mask[in] ? phi[in] : 0.0) - v.rob * phi[e];
    }
    if (kb < 0 || kb >= v.nz) return 0.0;
    const long n = i + (long)v.nx * (j + (long)v.ny * kb);
    return mask[n] ? phi[n] : 0.0;
}

// Cells whose field stencil (the 32 nodes of the differences at the eight corners) lies in
// the box, off the ghost planes, and on unknowns only: the gather reads phi as it stands.
__global__ void k_pic_open(PicView v, const uint8_t* __restrict__ mask, long ncell,
                           uint8_t* __restrict__ open) {
    const long c = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (c >= ncell) return;
    const int i = (int)(c % (v.nxl - 1));
    const long jk = c / (v.nxl - 1);
    const int j = (int)(jk % (v.nyl - 1)), kb = (int)(jk / (v.nyl - 1)) + v.zoff;
    const int g = v.rob > 0.0 ? 1 : 0;
    bool ok = i >= 1 && i + 2 < v.nx && j >= 1 && j + 2 < v.ny && kb - 1 >= g && kb + 2 < v.nz - g;
    if (ok) {
        for (int z = -1; z <= 2; ++z)
            for (int y = -1; y <= 2; ++y)
                for (int x = -1; x <= 2; ++x) {
                    const int out = (x < 0 || x > 1) + (y < 0 || y > 1) + (z < 0 || z > 1);
                    if (out < 2)
                        ok = ok && mask[i + x + (long)v.nx * (j + y + (long)v.ny * (kb + z))] != 0;
                }
    }
    open[c] = ok;
}

// Two neighbouring values of phi: one 16-byte load (8-byte alignment is enough for it).
typedef double PicPair __attribute__((ext_vector_type(2), aligned(8)));
__device__ inline PicPair pic_pair(const double* __restrict__ p) {
    return *reinterpret_cast<const PicPair*>(p);
}

// One thread per particle.  Bound by the lines its 32 nodes lie on: particles are in no
// order, so every lane of a load reads lines of its own, and 48 loads of phi and 48 of the
// mask a particle (each corner's differences by themselves) missed the first-level cache on
// most of them.  An open cell takes 16 loads of two neighbours, the two of a line next to
// each other, and no mask: 2 million particles on 192 x 192 x 1024 1121 -> 195 us.
__global__ __launch_bounds__(256) void k_pic_gather(PicView v, const double* __restrict__ phi,
                                                    const uint8_t* __restrict__ mask,
                                                    const uint8_t* __restrict__ open,
                                                    const double* __restrict__ pos, long n,
                                                    double* __restrict__ E) {
    const long p = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (p >= n) return;
    int ci, cj, ck;
    double fx, fy, fz;
    double ex = 0.0, ey = 0.0, ez = 0.0;
    if (pic_cell(v, pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], &ci, &cj, &ck, &fx, &fy, &fz)) {
        const int kb = ck + v.zoff;
        // [z][y][x] of the nodes: the lines along x, y and z through the cell's corners
        double lx[2][2][4], ly[2][4][2], lz[4][2][2];
        if (open[ci + (v.nxl - 1) * (cj + (long)(v.nyl - 1) * ck)]) {
            const long sy = v.nx, sz = sy * v.ny;
            const double* o = phi + ci + sy * cj + sz * kb;
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const double* a = o + y * sy + z * sz;
                    const PicPair l = pic_pair(a - 1), r = pic_pair(a + 1);
                    lx[z][y][0] = l.x;
                    lx[z][y][1] = l.y;
                    lx[z][y][2] = r.x;
                    lx[z][y][3] = r.y;
                }
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int y = 0; y < 4; y += 3) {
                    const PicPair a = pic_pair(o + (y - 1) * sy + z * sz);
                    ly[z][y][0] = a.x;
                    ly[z][y][1] = a.y;
                }
#pragma unroll
            for (int z = 0; z < 4; z += 3)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const PicPair a = pic_pair(o + y * sy + (z - 1) * sz);
                    lz[z][y][0] = a.x;
                    lz[z][y][1] = a.y;
                }
        } else {
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        lx[z][y][x] = pic_phi(v, phi, mask, ci - 1 + x, cj + y, kb + z);
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int y = 0; y < 4; y += 3)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        ly[z][y][x] = pic_phi(v, phi, mask, ci + x, cj - 1 + y, kb + z);
#pragma unroll
            for (int z = 0; z < 4; z += 3)
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        lz[z][y][x] = pic_phi(v, phi, mask, ci + x, cj + y, kb - 1 + z);
        }
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    ly[z][1 + y][x] = lx[z][y][1 + x];
                    lz[1 + z][y][x] = lx[z][y][1 + x];
                }
#pragma unroll
        for (int dz = 0; dz < 2; ++dz) {
            const double wz = dz ? fz : 1.0 - fz;
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
                const double wy = dy ? fy : 1.0 - fy;
#pragma unroll
                for (int dx = 0; dx < 2; ++dx) {
                    const double wx = dx ? fx : 1.0 - fx;
                    const double w = wx * wy * wz;
                    ex += w * (-(lx[dz][dy][dx + 2] - lx[dz][dy][dx]) / (2.0 * v.hx));
                    ey += w * (-(ly[dz][dy + 2][dx] - ly[dz][dy][dx]) / (2.0 * v.hy));
                    ez += w * (-(lz[dz + 2][dy][dx] - lz[dz][dy][dx]) / (2.0 * v.hz));
                }
            }
        }
    }
    E[3 * p] = ex;
    E[3 * p + 1] = ey;
    E[3 * p + 2] = ez;
}

static PicView pic_view(const saamg_pic* P) {
    PicView v;
    v.nx = P->g.nx;
    v.ny = P->g.ny;
    v.nz = P->g.nz;
    v.zoff = P->g.z_offset;
    v.nxl = P->nxl;
    v.nyl = P->nyl;
    v.nzl = P->nzl;
    v.ox = P->g.origin[0];
    v.oy = P->g.origin[1];
    v.oz = P->g.origin[2];
    v.hx = P->g.h[0];
    v.hy = P->g.h[1];
    v.hz = P->g.h[2];
    v.rob = (P->g.robin_d > 0.0 && P->g.z_offset == 1) ? 2.0 * P->g.h[2] / P->g.robin_d : 0.0;
    return v;
}

// Run sums are kept by cell where there are fewer cells than particles, else by the run's
// first particle: the smaller array.
static bool pic_by_cell(const saamg_pic* P) { return P->ncell < P->cap; }
static long pic_rows(const saamg_pic* P) { return (long)(P->nyl - 1) * (P->nzl - 1); }

void pic_workspace(long ncell, long nrow, long cap, size_t* run, size_t* carry, size_t* row) {
    *run = 64 * (size_t)std::min(ncell, cap);
    *carry = 64 * (size_t)((cap + kChunk - 1) / kChunk);
    *row = 4 * (size_t)(nrow + 1);
}

void pic_open(saamg_pic* P, hipStream_t s) {
    hipLaunchKernelGGL(k_pic_open, dim3((unsigned)((P->ncell + 255) / 256)), dim3(256), 0, s, pic_view(P),
                       P->mask, P->ncell, P->open);
    HIPCHECK(hipGetLastError());
}

void pic_deposit(saamg_pic* P, const double* pos, long n, double q, double* rho, hipStream_t s) {
    const PicView v = pic_view(P);
    const uint32_t sentinel = (uint32_t)P->ncell;
    if (n > 0) {
        hipLaunchKernelGGL(k_pic_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, v, pos, n,
                           sentinel, P->key, P->idx);
        HIPCHECK(hipGetLastError());
        size_t bytes = P->tmp_bytes;
        HIPCHECK(hipcub::DeviceRadixSort::SortPairs(P->tmp, bytes, P->key, P->key_s, P->idx, P->idx_s,
                                                    (int)n, 0, P->key_bits, s));
    }
    const long nrow = pic_rows(P), nchunk = (n + kChunk - 1) / kChunk;
    hipLaunchKernelGGL(k_pic_runs, dim3((unsigned)(nchunk + nrow / kChunk + 1)), dim3(kChunk), 0, s, v, pos,
                       P->key_s, P->idx_s, (int)n, (int)nchunk, sentinel, q, pic_by_cell(P), nrow, P->run,
                       P->carry, P->cell, P->row);
    HIPCHECK(hipGetLastError());
    const long nxy = (long)v.nx * v.ny, groups = (v.nz + kPicPlanes - 1) / kPicPlanes;
    hipLaunchKernelGGL(k_pic_nodes, dim3((unsigned)((nxy + 255) / 256), (unsigned)std::min(groups, 65535l)),
                       dim3(256), 0, s, v, P->key_s, P->row, P->cell, P->run, P->carry, pic_by_cell(P), rho);
    HIPCHECK(hipGetLastError());
}

void pic_gather(saamg_pic* P, const double* phi, const double* pos, long n, double* E, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_pic_gather, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pic_view(P),
                       phi, P->mask, P->open, pos, n, E);
    HIPCHECK(hipGetLastError());
}

size_t pic_sort_bytes(long n, int bits) {
    size_t bytes = 0;
    HIPCHECK(hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, (const uint32_t*)nullptr,
                                                (uint32_t*)nullptr, (const int32_t*)nullptr,
                                                (int32_t*)nullptr, (int)n, 0, bits, (hipStream_t)0));
    return bytes;
}

}  // namespace saamg
