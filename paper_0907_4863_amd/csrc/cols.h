// Device helpers of the level-0 kernels that keep stencil rows by column (the V-cycle's strokes
// and the CG passes): a wavefront owns 64 consecutive columns of 3 lines, one column per lane
// and line, and marches along z.
//
// A column's stencil row (the six neighbour coefficients; zeros where the node is not an
// unknown) is held in registers and read again only where a line differs from the line one
// plane below (FineLevel::zinfo), which a pipe of constant cross-section does at its ends only:
// a plane then needs no masks, slots or table rows, and every lane runs the same code whether
// its row is regular, irregular or empty.
#pragma once

#include "march.h"

namespace saamg {

template <typename T>
struct StrokeView {
    int nx, ny, nz, nsegx;
    long nxy;
    const uint64_t* unk;
    const uint64_t* irr;
    const int32_t* base;
    const T* tab;
    const T* tabT;
    T c[3];
    const uint8_t* zinfo;   // [ny][nz + 1], see k_zinfo
    const TileAt* tiles;    // the tiles of the cross-section that hold unknowns
    int live, S;            // their number; planes per slab (a multiple of 3)
    const double* skip;
};

// Stencil rows of a wavefront's 3 x 64 columns on one plane.
template <typename T, bool TR>
struct Cols {
    T a[3][6];
    T at[TR ? 3 : 1][6];  // rows of the transpose
    uint64_t um[3];       // the lanes whose node is an unknown
};

// What a line's entry of zinfo says (see k_zinfo).
constexpr int kSlotRow = -1, kSlotNone = -2;
constexpr int kZSame = 1, kZUnk = 2, kZRep = 2;  // bits, and the shift of 1 + (rep - z)

// Whole-wavefront shift by one lane with 0 from beyond the wavefront (lane l receives lane
// l - 1 (UP) or l + 1), in a form the compiler can fold into the consuming instruction.
template <bool UP>
__device__ __forceinline__ float shift0(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 UP ? 0x138 : 0x130, 0xf, 0xf, true));
}
template <bool UP>
__device__ __forceinline__ double shift0(double v) {
    const uint64_t s = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)s, UP ? 0x138 : 0x130, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(s >> 32), UP ? 0x138 : 0x130, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// One plane of a box vector as a bounds-checked buffer: a lane whose byte offset is kOff
// reads 0 and writes nothing, and so does every lane on a plane that is not there (ok
// false).  The march then needs no branch around its loads and stores.
constexpr unsigned kOff = 0x80000000u;
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane(const T* a, int bytes, bool ok) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)a, 0, ok ? bytes : 0, 0x00027000);
}
// The loaded values are first used here: keeps the compiler from moving the use (and the
// wait for the load) ahead of the barrier before it.
__device__ __forceinline__ float here(float v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ double here(double v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, unsigned o, float& v) {
    v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)o, 0, 0));
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, unsigned o, double& v) {
    v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)o, 0, 0));
}
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, unsigned o, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)o, 0, 0);
}
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, unsigned o, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)o, 0, 0);
}

// The rows in use along a slab.  Planes are counted from the slab's first, p0; up to 64.
// SP: the rows of the symmetric part, (A + A^T) / 2, in place of A's.
template <typename T, bool TR, bool SP = false>
struct Rows {
    Cols<T, TR> c;
    uint64_t change;  // planes whose rows differ from those of the plane below; bit 0 set
    uint64_t unk;     // planes with an unknown in the wavefront's columns' lines
    int info[3];      // zinfo of the lines at plane p0 + lane
    // Groups are numbered from the slab's first plane; a wavefront keeps the table slots of its
    // nodes (kSlotRow: the interior row, kSlotNone: not an unknown) for the last three groups
    // it met in LDS, because the stages, on three consecutive planes, go back and forth between
    // the groups where they change, and a row read again by its slot is one short trip to
    // the cache instead of three.
    int held = 0, newest = 0;
    int* ring;  // [3 groups][3 lines][64]
    // Planes i at which a pipeline of stages on planes i - first .. i - first - 2 runs with the
    // rows it holds: all of them, and the one before, share one group's rows and have unknowns.
    __device__ __forceinline__ uint64_t steady(int first) const {
        const uint64_t go = unk & (unk << 1) & (unk << 2) & (unk << 3) &
                            ~(change | (change << 1) | (change << 2));
        return go << first;
    }
    __device__ __forceinline__ void init(const StrokeView<T>& v, int yb, int p0) {
        const int z = p0 + (int)threadIdx.x;
        int all = kZSame | kZUnk, any = 0;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const int y = yb + l;
            info[l] = kZSame;
            if ((unsigned)y < (unsigned)v.ny && z >= 0 && z <= v.nz)
                info[l] = v.zinfo[(long)(v.nz + 1) * y + z];
            all &= info[l];
            any |= info[l];
        }
        change = ~__ballot(all & kZSame) | 1ull;
        unk = __ballot(any & kZUnk);
    }
    // Rows of plane i into c; false (and c unchanged) where the lines hold no unknown.  FAST:
    // on a steady plane they are there.
    template <bool FAST>
    __device__ __forceinline__ bool at(const StrokeView<T>& v, int x, int yb, int p0, int i) {
        if (FAST) return true;
        i = max(i, 0);
        if (!((unk >> i) & 1ull)) return false;
        const int g = (int)__popcll(change & ((2ull << i) - 1ull));
        if (g != held) {
            held = g;
            load(v, x, yb, p0, i, g);
        }
        return true;
    }
    // Table slots of the lines on plane i.
    struct Words {
        uint64_t u[3], r[3];
        int b0[3];
    };
    __device__ __forceinline__ Words words(const StrokeView<T>& v, int x, int yb, int p0, int i) {
        Words q;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const int inf = __builtin_amdgcn_readlane(info[l], i);
            const int y = yb + l, z = p0 + i + (inf >> kZRep) - 1;  // the plane that has the rows
            q.u[l] = q.r[l] = 0;
            q.b0[l] = 0;
            if ((inf & kZUnk) && (unsigned)x < (unsigned)v.nx) {
                const long s = ((long)z * v.ny + y) * v.nsegx + (x >> 6);
                q.u[l] = v.unk[s];
                q.r[l] = v.irr[s];
                q.b0[l] = v.base[s];
            }
        }
        return q;
    }
    static __device__ __forceinline__ int slot_of(const Words& q, int b, int l) {
        return !((q.u[l] >> b) & 1ull) ? kSlotNone
               : !((q.r[l] >> b) & 1ull) ? kSlotRow
                                         : q.b0[l] + (int)__popcll(q.r[l] & ((1ull << b) - 1ull));
    }
    // returns the lanes whose column holds an unknown
    __device__ __forceinline__ uint64_t keep(const Words& q, int x, int g) {
        int* e = ring + (g % 3) * 192 + threadIdx.x;
        bool u = false;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const int s = slot_of(q, x & 63, l);
            u = u || s != kSlotNone;
            e[64 * l] = s;
        }
        return __ballot(u);
    }
    // The slots of the first three groups of the n planes the slab's stages visit, read
    // together: their trips to memory overlap each other and the march's first planes.  False
    // when the columns of `out` (the lanes whose nodes the wavefront writes) hold no unknown.
    __device__ __forceinline__ bool preload(const StrokeView<T>& v, int x, int yb, int p0, int n,
                                            uint64_t out) {
        const uint64_t in = n < 64 ? (1ull << n) - 1ull : ~0ull;
        Words q[3];
        int gs[3];
        uint64_t left = unk & in;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            gs[k] = 0;
            if (left == 0) continue;  // wave-uniform
            const int i = (int)__builtin_ctzll(left);
            gs[k] = (int)__popcll(change & ((2ull << i) - 1ull));
            q[k] = words(v, x, yb, p0, i);
            // the planes beyond this group
            const uint64_t later = change & ~((2ull << i) - 1ull);
            left &= later ? ~((later & (0 - later)) - 1ull) : 0ull;
        }
        // the lines know their unknowns, not the columns: a wavefront whose columns hold none
        // (beside the pipe, most often) has no plane to work on
        bool all = left == 0;
        uint64_t some = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (gs[k] <= newest) continue;
            if (gs[k] >= gs[0] + 3) {
                all = false;
                continue;
            }
            some |= keep(q[k], x, gs[k]);
            newest = gs[k];
        }
        if (all && some == 0) unk = 0;
        return out != 0 && unk != 0 && (!all || (some & out) != 0);
    }
    __device__ __forceinline__ void load(const StrokeView<T>& v, int x, int yb, int p0, int i, int g) {
        if (g > newest) {  // the first stage meets the groups in order
            newest = g;
            (void)keep(words(v, x, yb, p0, i), x, g);
        }
        const int* e = ring + (g % 3) * 192 + threadIdx.x;
        const int slot[3] = {e[0], e[64], e[128]};
        fill(v, slot);
    }
    // The rows of the given slots.
    __device__ __forceinline__ void fill(const StrokeView<T>& v, const int (&slot)[3]) {
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            c.um[l] = __ballot(slot[l] != kSlotNone);
#pragma unroll
            for (int d = 0; d < 6; ++d) {
                c.a[l][d] = slot[l] != kSlotNone ? v.c[d >> 1] : T(0);
                if (TR) c.at[l][d] = c.a[l][d];
            }
            if (slot[l] >= 0) {
                load_row6(v.tab, (long)slot[l], 0u, c.a[l]);
                if (TR) load_row6(v.tabT, (long)slot[l], 0u, c.at[l]);
                if (SP) {
                    T t[6];
                    load_row6(v.tabT, (long)slot[l], 0u, t);
#pragma unroll
                    for (int d = 0; d < 6; ++d) c.a[l][d] = T(0.5) * (c.a[l][d] + t[d]);
                }
            }
        }
        // the rows have landed before the branch around this read ends, so that the common
        // path waits for none of them (nor, with them, for the planes in flight)
        settle(c.a);
        if (TR) settle(c.at);
    }
    // For a march with a single stencil, which takes the planes in order: rows of plane i
    // (false: the lines hold no unknown there).
    __device__ __forceinline__ bool next(const StrokeView<T>& v, int x, int yb, int p0, int i) {
        if (!((unk >> i) & 1ull)) return false;
        if ((change >> i) & 1ull) {
            const Words q = words(v, x, yb, p0, i);
            int slot[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) slot[l] = slot_of(q, x & 63, l);
            fill(v, slot);
        }
        return true;
    }
};

// (A X) on the three lines of a wavefront: own lines c, the planes below and above, the
// lines before and after (ylo, yhi).
template <typename T>
__device__ __forceinline__ void apply3(const T (&a)[3][6], const T (&c)[3], const T (&zm)[3],
                                       const T (&zp)[3], T ylo, T yhi, T (&o)[3]) {
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const T ym = l ? c[l - 1] : ylo, yp = l < 2 ? c[l + 1] : yhi;
        o[l] = c[l] + shift0<true>(c[l]) * a[l][0] + shift0<false>(c[l]) * a[l][1] + a[l][2] * ym +
               a[l][3] * yp + a[l][4] * zm[l] + a[l][5] * zp[l];
    }
}

// Tile of a block (the live tiles along x, then y, then slabs; neighbours in this order share
// an XCD's L2: each XCD takes a run of consecutive tiles).
template <typename T>
__device__ __forceinline__ void stroke_tile(const StrokeView<T>& v, int* tx, int* ty, int* sz) {
    const unsigned b = blockIdx.x, nb = gridDim.x, q = nb >> 3;
    const unsigned lb = (b < 8 * q) ? (b & 7) * q + (b >> 3) : b;
    const TileAt t = v.tiles[lb % (unsigned)v.live];
    *tx = t.x;
    *ty = t.y;
    *sz = (int)(lb / (unsigned)v.live);
}

}  // namespace saamg
