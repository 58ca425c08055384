// Patch recurrence kernels of libsq for gfx950: FP64 Lanczos bounds and Chebyshev
// moments (SQDFT, arXiv 1708.07913, Sec. 3.2-3.3) on cubes of 25 to 31 points whose projector spheres do not overlap.
//
// One workgroup works on one region of influence at a time; a thread owns a
// patch of 2 x 2 cube columns and sweeps the planes upward:
//   * the x and y legs of the stencil come from an LDS copy of the plane, read
//     as aligned x pairs (16-byte reads reach 275 B per cycle and CU, pairs of
//     8-byte reads in one instruction 138): 12 words per point, in batches of six
//     pairs that are issued one batch ahead of their use;
//   * the z legs come from a register window of 2 NO + 1 planes;
//   * the vector itself stays in registers (mostly accumulation registers, where
//     the compiler puts what the vector ALU does not need at once), plane by
//     plane in place of the previous one;
//   * the previous vector streams through the workgroup's slot; its first planes
//     stay in LDS.
//
// Projectors: where no two spheres overlap, every grid point belongs to at most
// one of them; its projector value is read from a periodic grid like V_eff, and
// a byte per cube point (LDS) names the region's image.  A point outside every
// sphere has the value 0 and may carry any label.
#ifndef SQ_KEEP_BRANCH_ENDS
#error "compile with -mllvm -amdgpu-remove-redundant-endcf=0 -DSQ_KEEP_BRANCH_ENDS (see TILE_FLAGS in build.py for why)"
#endif
#include "sq_device.h"

#include <type_traits>

namespace sq {
namespace {

constexpr int NO = kNoMax;
constexpr int kLdsBytes = 160 * 1024;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int pair_stride(int lanes) {
    int pe = lanes + NO / 2;
    while ((2 * pe - lanes) % 16) ++pe;
    return pe;
}

template <int C>
struct Tile {
    static constexpr int RY = kPatchRows;           // y-adjacent points of a thread (two x-adjacent ones)
    static constexpr int NP = 2 * RY;               // points of a thread in a plane
    static constexpr int XW = patch_lanes(C);       // threads along x
    static constexpr int YG = (C + RY - 1) / RY;    // threads along y
    static constexpr int NT = XW * YG;
    static constexpr unsigned SPLANE = (unsigned)(RY * patch_block(C)) * 16u;  // bytes of a slot plane
    static constexpr int BLOCK = patch_block(C);
    static constexpr int CC = C * C;
    // Plane copy: a row for every thread row and 2 NO halo rows of PE x pairs,
    // NO / 2 zero pairs before each row's values; a row's right halo is the next
    // row's left one.
    // PE keeps consecutive threads in consecutive bank groups across thread rows
    // (2 PE = XW modulo the 16 groups of a 16-byte access; 19 pairs a row cost
    // half the LDS rate).
    static constexpr int PE = pair_stride(XW);
    static constexpr int YALL = (BLOCK + XW - 1) / XW * RY;  // rows of all threads, idle ones included
    static constexpr int ROWS = YALL + 2 * NO;
    static constexpr int PLANE = 2 * (ROWS * PE + NO);
    static constexpr int NBUF = 3;
    static constexpr int LW = 2 * ((C + 1) / 2);    // label row
    static constexpr int LABZ = C * LW;
    static constexpr int LAB = C * LABZ + ((YALL - C + 1) * LW + 2 * XW + 3) / 4 * 4;  // with slack for idle threads
    static constexpr int IPT = (kMaxImages + BLOCK - 1) / BLOCK;  // images per thread
    static_assert(C % 2 == 1 && 2 * XW > C && NT <= BLOCK, "patches cover the cube");
};

template <int C>
struct TileTables {
    double s[kMaxImages];      // projector dots of the vector being formed
    double cs[kMaxImages];     // scaled coefficients of the projector term
    alignas(16) double plane[Tile<C>::NBUF][Tile<C>::PLANE];
    double red[4 * 8];
    double bc[4];
    int img_atom[kMaxImages];
    int img_lb[kMaxImages][3];
    int img_prefix[kMaxImages + 1];
    int ni, nruns, item, pad;
    alignas(4) unsigned char lab[Tile<C>::LAB];
};

// Planes of the previous vector that fit in LDS beside the tables (`extra`:
// bytes of a kernel's own tables).
template <int C>
constexpr int lds_planes(int extra) {
    const int room = (kLdsBytes - extra - 256 - (int)sizeof(TileTables<C>)) / (Tile<C>::NP * Tile<C>::BLOCK * 8);
    return room < 0 ? 0 : (room > C ? C : room);
}

template <int C, int NPL>
struct TileLds : TileTables<C> {
    alignas(16) double2 prev[NPL > 0 ? NPL : 1][Tile<C>::RY][Tile<C>::BLOCK];
};

// Sum over the 64 lanes: neighbours within 16 lanes by DPP, then the four
// groups' sums through scalar registers (uniform result).
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_uniform(double v) {
    v = dpp_add<0xB1>(v);   // lanes ^ 1
    v = dpp_add<0x4E>(v);   // lanes ^ 2
    v = dpp_add<0x141>(v);  // mirrored within 8
    v = dpp_add<0x140>(v);  // mirrored within 16
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// A thread's points of a plane in the workgroup's slot: 16-byte accesses,
// contiguous over the workgroup; `voff` per patch row, `soff` of the plane.
template <int RY>
__device__ __forceinline__ void slot_read(__amdgpu_buffer_rsrc_t r, const unsigned (&voff)[RY], unsigned soff,
                                          double (&v)[2 * RY]) {
#pragma unroll
    for (int h = 0; h < RY; ++h) {
        const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(r, voff[h], soff, 0);
        v[2 * h] = __builtin_bit_cast(double, u32x2{b.x, b.y});
        v[2 * h + 1] = __builtin_bit_cast(double, u32x2{b.z, b.w});
    }
}
template <int RY>
__device__ __forceinline__ void slot_write(__amdgpu_buffer_rsrc_t r, const unsigned (&voff)[RY], unsigned soff,
                                           const double (&v)[2 * RY]) {
#pragma unroll
    for (int h = 0; h < RY; ++h) {
        const u32x2 a = __builtin_bit_cast(u32x2, v[2 * h]), b = __builtin_bit_cast(u32x2, v[2 * h + 1]);
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{a.x, a.y, b.x, b.y}, r, voff[h], soff, 0);
    }
}

// a += k v as one 4-byte instruction.  (Left to contract a += k * v by itself,
// the compiler shares the product k v between the two points that need it and
// spends a multiplication and two 8-byte additions on them.)
__device__ __forceinline__ void fma_to(double &a, double k, double v) { a = __builtin_fma(k, v, a); }

// Keeps values materialised together (see pin).
__device__ __forceinline__ void pin_all(double (&x)[2]) { asm volatile("" : "+v"(x[0]), "+v"(x[1])); }
__device__ __forceinline__ void pin_all(double (&x)[4]) {
    asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
}

// A thread's place in the cube; point r of its patch is (x + r % 2, y + r / 2).
template <int C>
struct Place {
    using T = Tile<C>;
    int x, y;       // threads past the cube hold zeros
    unsigned cell;  // LDS index of point 0 in the plane copy
    unsigned loff;  // label offset of point 0
    unsigned slot[T::RY];  // byte offsets in a slot plane
    __device__ __forceinline__ void init(int tid) {
        x = 2 * (tid % T::XW);
        y = tid / T::XW * T::RY;
        cell = (unsigned)(2 * ((y + NO) * T::PE + NO / 2) + x);
        loff = (unsigned)(y * T::LW + x);
#pragma unroll
        for (int h = 0; h < T::RY; ++h) slot[h] = (unsigned)(h * T::BLOCK + tid) * 16u;
    }
    __device__ __forceinline__ bool valid(int r) const { return x + (r & 1) < C && y + (r >> 1) < C; }
};

// Images whose spheres meet the cube of node (qi, qj, qk), and their labels.
template <int C, typename AT, typename LdsT>
__device__ void tile_setup(const AT &A, LdsT &L, int qi, int qj, int qk, int tid) {
    const int n = A.n, m = A.m;
    __syncthreads();
    if (tid == 0) {
        L.ni = 0;
        L.nruns = 0;
    }
    for (int i = tid; i < kMaxImages; i += Tile<C>::BLOCK) L.s[i] = L.cs[i] = 0.0;
    for (int i = tid; i < Tile<C>::LAB / 4; i += Tile<C>::BLOCK)
        reinterpret_cast<unsigned *>(&L.lab[0])[i] = ~0u;
    __syncthreads();
    const int lo0 = qi - m, lo1 = qj - m, lo2 = qk - m;
    for (int a = tid; a < A.natom; a += Tile<C>::BLOCK) {
        const AtomDev at = A.atoms[a];
        const int tl0 = ceil_div(lo0 - at.bx - at.dmax[0], n), th0 = floor_div(lo0 + C - 1 - at.bx - at.dmin[0], n);
        const int tl1 = ceil_div(lo1 - at.by - at.dmax[1], n), th1 = floor_div(lo1 + C - 1 - at.by - at.dmin[1], n);
        const int tl2 = ceil_div(lo2 - at.bz - at.dmax[2], n), th2 = floor_div(lo2 + C - 1 - at.bz - at.dmin[2], n);
        for (int tz = tl2; tz <= th2; ++tz)
            for (int ty = tl1; ty <= th1; ++ty)
                for (int tx = tl0; tx <= th0; ++tx) {
                    const int slot = atomicAdd(&L.ni, 1);
                    if (slot < kMaxImages) {
                        L.img_atom[slot] = a;
                        L.img_lb[slot][0] = at.bx + n * tx - lo0;
                        L.img_lb[slot][1] = at.by + n * ty - lo1;
                        L.img_lb[slot][2] = at.bz + n * tz - lo2;
                        L.img_prefix[slot + 1] = at.nrun;
                    }
                }
    }
    __syncthreads();
    // uniform by construction and to the compiler: the barriers below stand in no
    // branch that it would lower with an execution mask
    int ni = __builtin_amdgcn_readfirstlane(L.ni);
    if (ni > kMaxImages) {
        if (tid == 0) atomicOr(A.flags, kFlagImages);
        ni = kMaxImages;
    }
    if (tid == 0) {
        int acc = 0;
        L.img_prefix[0] = 0;
        for (int i = 0; i < ni; ++i) {
            acc += L.img_prefix[i + 1];
            L.img_prefix[i + 1] = acc;
        }
    }
    __syncthreads();
    const int npairs = __builtin_amdgcn_readfirstlane(L.img_prefix[ni]);
    int count = 0;
    for (int p = tid; p < npairs; p += Tile<C>::BLOCK) {
        int lo = 0, hi = ni;  // largest I with prefix[I] <= p
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (L.img_prefix[mid] <= p) lo = mid;
            else hi = mid;
        }
        const int I = lo;
        const RunDev rr = A.runs[A.atoms[L.img_atom[I]].run0 + (p - L.img_prefix[I])];
        const int cx = L.img_lb[I][0] + rr.dx, cy = L.img_lb[I][1] + rr.dy;
        if (cx < 0 || cx >= C || cy < 0 || cy >= C) continue;
        const int z0 = L.img_lb[I][2] + rr.dz0, z1 = z0 + rr.len - 1;
        if (z0 >= C || z1 < 0) continue;
        ++count;
        const int zl = z0 > 0 ? z0 : 0, zh = z1 < C - 1 ? z1 : C - 1;
        unsigned char *dst = &L.lab[cy * Tile<C>::LW + cx];
        for (int z = zl; z <= zh; ++z) dst[z * Tile<C>::LABZ] = (unsigned char)I;
    }
    if (count) atomicAdd(&L.nruns, count);
    __syncthreads();
    if (tid == 0 && L.nruns > max_region_runs(C)) atomicOr(A.flags, kFlagRuns);
    // points outside every sphere take the label of the next run above them, so
    // that a column changes its label once per run (left out where all 256
    // labels name images)
    if (ni < kMaxImages) {
        for (int col = tid; col < Tile<C>::CC; col += Tile<C>::BLOCK) {
            unsigned char *p = &L.lab[col / C * Tile<C>::LW + col % C];
            unsigned l[C];
#pragma unroll
            for (int z = 0; z < C; ++z) l[z] = p[z * Tile<C>::LABZ];
            unsigned last = 255u, first = 255u;
#pragma unroll
            for (int z = 0; z < C; ++z) {
                if (l[z] != 255u) last = l[z];
            }
            first = last;
#pragma unroll
            for (int z = C - 1; z >= 0; --z) {
                if (l[z] != 255u) first = l[z];
                p[z * Tile<C>::LABZ] = (unsigned char)first;
            }
        }
        __syncthreads();
    }
}

// What a sweep does with the vector t it reads and the vector it forms:
//   kMoments  t^{k+1} = so (H t^k) - t^{k-1} + projector term
//   kLanczos  x_j = u_{j-1} - fa x_{j-1} formed ahead of the stencil, then
//             u_j = so (H' x_j) - fb x_{j-1} + projector term
enum SweepMode { kMoments, kLanczos };

struct SweepArgs {
    double so;      // scale of the local part
    double fa, fb;  // Lanczos formation coefficients
    double c0;      // diagonal added to V_eff
    bool prev;      // the previous vector exists (otherwise its slot is not read)
};

// A thread's points of the current vector (the previous one is in LDS and the slot).
template <int C>
struct Vec {
    double v[C][Tile<C>::NP];
};
template <int MODE, int C, int NPL, typename LdsT>
__device__ __forceinline__ void tile_sweep(LdsT &L, const Place<C> &pl, Vec<C> &X, const double (&kw)[NO + 1],
                                           __amdgpu_buffer_rsrc_t slr, __amdgpu_buffer_rsrc_t vr,
                                           __amdgpu_buffer_rsrc_t pr, const unsigned (&vcol)[Tile<C>::NP],
                                           unsigned zbase, int n, const SweepArgs &st, int tid, double (&dd)[2],
                                           double &centre) {
    using T = Tile<C>;
    constexpr int NP = T::NP, RY = T::RY, CC = T::CC, MC = (C - 1) / 2, WN = 2 * NO + 2, PE = T::PE;
    constexpr bool kForm = MODE == kLanczos;
    double W[WN][NP];        // planes z - NO .. z + NO + 1 of the vector
    double acc[NP], cz[NP];  // running projector dots, coefficients of the current labels
    unsigned lc[NP], ln[NP];
    double vz[NP], pz[NP];
    // the previous vector: planes of both parities, loaded two planes ahead (pw: the
    // current plane's, loaded again for kLanczos)
    double pv[2][NP], pw[NP];
    unsigned rslot[RY];
#pragma unroll
    for (int h = 0; h < RY; ++h) rslot[h] = st.prev ? pl.slot[h] : kIdleOffset;
    // running slot offsets (opaque, so that no table of them is kept in registers)
    unsigned rat = NPL * T::SPLANE, wat = rat, pat = rat;
    asm volatile("" : "+s"(rat), "+s"(wat), "+s"(pat));
    // byte offset of the current plane in the periodic grids
    const unsigned vstep = (unsigned)(n * n) * 8u, vend = vstep * (unsigned)n;
    unsigned vat = (unsigned)__builtin_amdgcn_readfirstlane((int)(zbase * vstep));
    asm volatile("" : "+s"(vat));
    auto load_potential = [&]() {
#pragma unroll
        for (int r = 0; r < NP; ++r) vz[r] = bload<double>(vr, vcol[r], vat);
    };
    auto load_values = [&]() {
#pragma unroll
        for (int r = 0; r < NP; ++r) pz[r] = bload<double>(pr, vcol[r], vat);
        vat += vstep;
        if (vat == vend) vat = 0;
    };
    auto read_prev = [&](int z, unsigned &at, double(&v)[NP]) {
        if (z < NPL) {
#pragma unroll
            for (int h = 0; h < RY; ++h) {
                const double2 d = L.prev[z][h][tid];
                v[2 * h] = d.x;
                v[2 * h + 1] = d.y;
            }
        } else {
            slot_read<RY>(slr, rslot, at, v);
            at += T::SPLANE;
        }
    };
    auto load_prev = [&](int z) { read_prev(z, rat, pv[z % 2]); };
    auto store_prev = [&](int z, const double(&q)[NP]) {
        if (z < NPL) {
#pragma unroll
            for (int h = 0; h < RY; ++h) L.prev[z][h][tid] = make_double2(q[2 * h], q[2 * h + 1]);
        } else {
            slot_write<RY>(slr, pl.slot, wat, q);
            wat += T::SPLANE;
        }
    };
    auto labels = [&](int z, unsigned(&l)[NP]) {
#pragma unroll
        for (int r = 0; r < NP; ++r) l[r] = L.lab[pl.loff + (unsigned)(z * T::LABZ + (r >> 1) * T::LW + (r & 1))];
    };
    // plane z into the register window
    auto enter = [&](int z) {
        if constexpr (kForm) {
            // pv: x_{j-1} of this plane
#pragma unroll
            for (int r = 0; r < NP; ++r) W[z % WN][r] = X.v[z][r] - st.fa * pv[z % 2][r];
        } else {
#pragma unroll
            for (int r = 0; r < NP; ++r) W[z % WN][r] = X.v[z][r];
        }
    };
    auto publish = [&](int z) {
#pragma unroll
        for (int py = 0; py < RY; ++py)
            *reinterpret_cast<double2 *>(&L.plane[z % T::NBUF][pl.cell + (unsigned)(2 * py * PE)]) =
                make_double2(W[z % WN][2 * py], W[z % WN][2 * py + 1]);
    };
    // A batch holds six neighbouring x pairs, b < RY: pairs -3 .. -1 and
    // 1 .. 3 of patch row b; then the six rows below the patch and the six above it.
    constexpr int NB = RY + 2;
    double2 q[2][NO];
    double a[NP];
    auto batch = [&](int z, int b) {
        const double *p = &L.plane[z % T::NBUF][pl.cell];
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const int off = b < RY ? 2 * (b * PE + (i < 3 ? i - 3 : i - 2))
                                   : 2 * PE * (b == RY ? -1 - i : RY + i);
            q[(z * NB + b) % 2][i] = *reinterpret_cast<const double2 *>(p + off);
        }
    };
    // adds a batch's legs (and, with the rows above, those within the patch)
    auto legs = [&](int z, int b) {
        const double2(&o)[NO] = q[(z * NB + b) % 2];
        const double(&t)[NP] = W[z % WN];
        if (b < RY) {
            // the row's values by x offset from the thread's even point, -6 .. 7
            const double v[14] = {o[0].x, o[0].y, o[1].x, o[1].y, o[2].x, o[2].y, t[2 * b],
                                  t[2 * b + 1], o[3].x, o[3].y, o[4].x, o[4].y, o[5].x, o[5].y};
#pragma unroll
            for (int d = NO; d >= 1; --d)
#pragma unroll
                for (int px = 0; px < 2; ++px) {
                    // (the pair's own two come last)
                    if (d > 1 || px == 1) fma_to(a[2 * b + px], kw[d], v[6 + px + d]);
                    if (d > 1 || px == 0) fma_to(a[2 * b + px], kw[d], v[6 + px - d]);
                }
        } else if (b == RY) {
            // row i + 1 below patch row 0
#pragma unroll
            for (int i = NO - 1; i >= 0; --i)
#pragma unroll
                for (int py = 0; py < RY; ++py) {
                    if (py + i + 1 > NO) continue;
                    fma_to(a[2 * py], kw[py + i + 1], o[i].x);
                    fma_to(a[2 * py + 1], kw[py + i + 1], o[i].y);
                }
        } else {
            // row i above patch row RY - 1, then the patch's own neighbours
#pragma unroll
            for (int i = NO - 1; i >= 0; --i)
#pragma unroll
                for (int py = 0; py < RY; ++py) {
                    const int d = RY + i - py;
                    if (d > NO) continue;
                    fma_to(a[2 * py], kw[d], o[i].x);
                    fma_to(a[2 * py + 1], kw[d], o[i].y);
                }
#pragma unroll
            for (int r = 0; r < NP; ++r) {
                fma_to(a[r], kw[1], t[(r + 2) % NP]);
                fma_to(a[r], kw[1], t[r ^ 1]);
            }
        }
    };
    // z neighbours at distance d
    auto legs_z = [&](int z, int d) {
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            if (z + d < C) fma_to(a[r], kw[d], W[(z + d) % WN][r]);
            if (z - d >= 0) fma_to(a[r], kw[d], W[(z - d + WN) % WN][r]);
        }
    };

    load_potential();
    load_values();
    load_prev(0);
    load_prev(1);
#pragma unroll
    for (int z = 0; z <= NO; ++z) {
        enter(z);
        if constexpr (kForm) load_prev(z + 2);
    }
    if constexpr (kForm) read_prev(0, pat, pw);
    publish(0);
    publish(1);
#pragma unroll
    for (int r = 0; r < NP; ++r) acc[r] = 0.0;
    labels(0, lc);
    __syncthreads();  // planes 0 and 1; the projector coefficients
    batch(0, 0);
    labels(1, ln);
#pragma unroll
    for (int r = 0; r < NP; ++r) cz[r] = L.cs[lc[r]];
#pragma unroll
    for (int z = 0; z < C; ++z) {
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();  // plane z + 1
        const double(&t)[NP] = W[z % WN];
        if (z + 2 < C) publish(z + 2);
        // The sum of a point grows from the smallest terms on: far legs first within each
        // batch, the nearest ones at the end, the diagonal last.  One chain of 40 terms
        // that starts with the diagonal has 1.2-1.5 times the rounding error of the ring
        // kernels' tree of pair sums (and 2.4 times where V_eff is deep); in this order it
        // has the same.  (Zeros behind the pin keep the chain's start here; a first
        // product moved into the batches spilled.)
#pragma unroll
        for (int r = 0; r < NP; ++r) a[r] = 0.0;
        pin_all(a);
        double dv[NP];
#pragma unroll
        for (int r = 0; r < NP; ++r) dv[r] = (vz[r] + st.c0) * t[r];
        if (z + 1 < C) load_potential();
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            // the next batch is in flight while this one is added
            if (b + 1 < NB) batch(z, b + 1);
            else if (z + 1 < C) batch(z + 1, 0);
#pragma unroll
            for (int d = NO - b * NO / NB; d > NO - (b + 1) * NO / NB; --d) legs_z(z, d);
            legs(z, b);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < NP; ++r) a[r] += dv[r];
        double out[NP];
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            const double so = pl.valid(r) ? st.so : 0.0;
            if constexpr (kForm) out[r] = so * a[r] - st.fb * pw[r];
            else out[r] = so * a[r] - pv[z % 2][r];
        }
        if constexpr (kForm) {
            if (z + 1 < C) read_prev(z + 1, pat, pw);
        } else {
            if (z + 2 < C) load_prev(z + 2);
        }
#pragma unroll
        for (int r = 0; r < NP; ++r) out[r] += cz[r] * pz[r];
        if (z == MC) centre = out[(MC % 2) + 2 * (MC % RY)];
#pragma unroll
        for (int r = 0; r < NP; ++r) X.v[z][r] = out[r];
#pragma unroll
        for (int r = 0; r < NP; ++r) acc[r] += pz[r] * out[r];
        if (z + 1 < C) load_values();
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            dd[0] += out[r] * out[r];
            dd[1] += out[r] * t[r];
        }
        pin_all(dd);
        store_prev(z, t);
        if (z + NO + 1 < C) {
            enter(z + NO + 1);
            if constexpr (kForm) {
                if (z + NO + 3 < C) load_prev(z + NO + 3);
            }
        }
        // runs that end at this plane add their dot products
#pragma unroll
        for (int r = 0; r < NP; ++r) {
            if (z + 1 < C) {
                if (lc[r] != ln[r]) {
                    atomicAdd(&L.s[lc[r]], acc[r]);
                    acc[r] = 0.0;
                    cz[r] = L.cs[ln[r]];
                }
                lc[r] = ln[r];
            } else if (acc[r] != 0.0) {
                atomicAdd(&L.s[lc[r]], acc[r]);
            }
        }
        if (z + 2 < C) labels(z + 2, ln);
    }
}

template <int C, typename AT>
__device__ __forceinline__ void tile_columns(const AT &A, const Place<C> &pl, int qi, int qj,
                                             unsigned (&vcol)[Tile<C>::NP]) {
#pragma unroll
    for (int r = 0; r < Tile<C>::NP; ++r)
        vcol[r] = pl.valid(r) ? (unsigned)(pmod(qi - A.m + pl.x + (r & 1), A.n) +
                                           A.n * pmod(qj - A.m + pl.y + (r >> 1), A.n)) * 8u
                              : kIdleOffset;
}

// Sums of N values over the workgroup: one barrier; every thread adds the
// waves' sums in the same order.
template <int N, int C, typename LdsT>
__device__ __forceinline__ void tile_sum(LdsT &L, double (&v)[N], int tid) {
    constexpr int NW = Tile<C>::BLOCK / 64;
    static_assert(N <= 4 && NW <= 8, "per-wave reduction slots");
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = wave_sum_uniform(v[i]);
    if ((tid & 63) == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) L.red[8 * i + w] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double s = L.red[8 * i];
#pragma unroll
        for (int k = 1; k < NW; ++k) s += L.red[8 * i + k];
        v[i] = uniform(s);
    }
}

// Set-up shared by the kernels: the launch-wide part of LDS.
template <int C, typename LdsT>
__device__ __forceinline__ void tile_begin(LdsT &L, int tid) {
    for (int i = tid; i < Tile<C>::NBUF * Tile<C>::PLANE; i += Tile<C>::BLOCK) (&L.plane[0][0])[i] = 0.0;
}
template <int C, int NPL, typename LdsT>
__device__ __forceinline__ void clear_prev(LdsT &L, int tid) {
#pragma unroll
    for (int z = 0; z < NPL; ++z)
#pragma unroll
        for (int h = 0; h < Tile<C>::RY; ++h) L.prev[z][h][tid] = make_double2(0.0, 0.0);
}
// x_{j-1} or t^{k-1} at plane z, outside a sweep
template <int C, int NPL, typename LdsT>
__device__ __forceinline__ void prev_plane(const LdsT &L, const Place<C> &pl, __amdgpu_buffer_rsrc_t slr, int z,
                                           double (&v)[Tile<C>::NP], int tid) {
    constexpr int RY = Tile<C>::RY;
    if (z < NPL) {
#pragma unroll
        for (int h = 0; h < RY; ++h) {
            const double2 q = L.prev[z][h][tid];
            v[2 * h] = q.x;
            v[2 * h + 1] = q.y;
        }
    } else {
        slot_read<RY>(slr, pl.slot, (unsigned)z * Tile<C>::SPLANE, v);
    }
}
// Coefficients of the images tid, tid + BLOCK, ...
template <int C, typename AT, typename LdsT>
__device__ __forceinline__ void image_coefs(const AT &A, const LdsT &L, double (&coef)[Tile<C>::IPT], int tid) {
#pragma unroll
    for (int i = 0; i < Tile<C>::IPT; ++i) {
        const int I = tid + i * Tile<C>::BLOCK;
        coef[i] = I < L.ni && I < kMaxImages ? A.atoms[L.img_atom[I]].coef : 0.0;
    }
}
// cs = scale coef s and s cleared (between a sweep's last barrier and the next
// one's first).
template <int C, typename LdsT>
__device__ __forceinline__ void next_coefs(LdsT &L, const double (&coef)[Tile<C>::IPT], double scale, int tid) {
#pragma unroll
    for (int i = 0; i < Tile<C>::IPT; ++i) {
        const int I = tid + i * Tile<C>::BLOCK;
        if (I < kMaxImages) {
            L.cs[I] = scale * coef[i] * L.s[I];
            L.s[I] = 0.0;
        }
    }
}
// The thread that owns the cube's centre, and its point there.
template <int C>
constexpr int centre_tid() { return (C - 1) / 2 / Tile<C>::RY * Tile<C>::XW + (C - 1) / 4; }
template <int C>
constexpr int centre_point() { return (C - 1) / 2 % 2 + 2 * ((C - 1) / 2 % Tile<C>::RY); }

// t^0 = e_q and the projector coefficients of the first step (published by the
// sweep's first barrier).
template <int C, int NPL, typename AT, typename LdsT>
__device__ __forceinline__ void unit_vector(const AT &A, LdsT &L, Vec<C> &X, long long q, double invz, int tid) {
    using T = Tile<C>;
    constexpr int MC = (C - 1) / 2;
#pragma unroll
    for (int z = 0; z < C; ++z)
#pragma unroll
        for (int r = 0; r < T::NP; ++r)
            X.v[z][r] = z == MC && r == centre_point<C>() && tid == centre_tid<C>() ? 1.0 : 0.0;
    clear_prev<C, NPL>(L, tid);
    if (tid == 0) {
        const double p = A.pgrid[q];  // p_I . e_q
        if (p != 0.0) {
            const int I = L.lab[MC * T::LABZ + MC * T::LW + MC];
            L.cs[I] = invz * A.atoms[L.img_atom[I]].coef * p;
        }
    }
}

// ---------------------------------------------------------------------------
// Chebyshev moments.  29-point cubes, 256 workgroups: 25.7 us a step (ring kernel
// 35.3), 2040 cycles a plane.  Of a wave's cycles 45 % issue vector instructions (about
// 175 FP64 ones a plane), 10 % LDS and 9 % other instructions, 22 % wait for LDS, memory
// and the barrier and 14 % for an instruction's turn: with 512 registers a SIMD holds
// one wave, which hides only what the batches hide.
// ---------------------------------------------------------------------------
template <int C>
__global__ __launch_bounds__(Tile<C>::BLOCK, 1) void moments_tile_kernel(LaunchArgs K) {
    using T = Tile<C>;
    constexpr int NPL = lds_planes<C>(0);
    __shared__ TileLds<C, NPL> L;
    const int tid = threadIdx.x;
    Place<C> pl;
    pl.init(tid);
    tile_begin<C>(L, tid);
    const __amdgpu_buffer_rsrc_t slr =
        make_rsrc(reinterpret_cast<double *>(K.slots) + (long long)blockIdx.x * K.slot_elems, K.slot_elems * 8);

    WorkSource work;
    SnapPtr Ap;
    long long qfirst, qend, qstep;
    while (work.next(K, L, tid, Ap, qfirst, qend, qstep)) {
        const auto &A = *Ap;
        const int n = A.n, npl = A.npl, half = npl / 2;
        const __amdgpu_buffer_rsrc_t vr = make_rsrc(A.veff, A.nd * 8);
        const __amdgpu_buffer_rsrc_t pr = make_rsrc(A.pgrid, A.nd * 8);
        double kw[NO + 1];
        kw[0] = 0.0;
#pragma unroll
        for (int d = 1; d <= NO; ++d) kw[d] = uniform(-0.5 * A.w[d]);

        for (long long q = qfirst; q < qend; q += qstep) {
            int qi, qj, qk;
            node_coords(q, n, qi, qj, qk);
            tile_setup<C>(A, L, qi, qj, qk, tid);
            const unsigned zbase = (unsigned)pmod(qk - A.m, n);
            const double chi = uniform(A.chi[q]), invz = uniform(1.0 / A.zeta[q]);
            unsigned vcol[T::NP];
            tile_columns<C>(A, pl, qi, qj, vcol);
            double *mrow = A.moments + q * (long long)(npl + 1);
            if (tid == 0) mrow[0] = 1.0;
            SweepArgs st;
            st.c0 = uniform(-3.0 * A.w[0] - chi);
            double coef[T::IPT];
            image_coefs<C>(A, L, coef, tid);
            Vec<C> X;
            unit_vector<C, NPL>(A, L, X, q, invz, tid);
            for (int k = 0; k < half; ++k) {
                st.so = k == 0 ? invz : 2.0 * invz;
                st.prev = k > 0;
                double d[2] = {0.0, 0.0}, centre = 0.0;
                tile_sweep<kMoments, C, NPL>(L, pl, X, kw, slr, vr, pr, vcol, zbase, n, st, tid, d, centre);
                if (tid == centre_tid<C>()) {
                    mrow[k + 1] = centre;
                    if (k == 0) L.bc[2] = centre;
                    if (fabs(centre) > 1.0 + A.bounds_tol) atomicOr(A.flags, kFlagBounds);
                }
                tile_sum<2, C>(L, d, tid);
                next_coefs<C>(L, coef, 2.0 * invz, tid);
                if (k + 1 > half / 2 && tid == 0) {
                    const double r2k = 2.0 * d[0] - 1.0, r2k1 = 2.0 * d[1] - L.bc[2];
                    mrow[2 * (k + 1)] = r2k;
                    mrow[2 * (k + 1) - 1] = r2k1;
                    if (fabs(r2k) > 1.0 + A.bounds_tol || fabs(r2k1) > 1.0 + A.bounds_tol)
                        atomicOr(A.flags, kFlagBounds);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Lanczos bounds, one sweep per step.  x_j = beta_{j-1} v_j is kept
// unnormalised (x_0 = v_0, the start vector), sigma_j = 1 / beta_{j-1}, and the
// sweep works with H' = H - s_j, s_j = alpha_{j-1}:
//   x_j = u_{j-1} - alpha' sigma_{j-1} x_{j-1}       (formed NO + 1 planes ahead)
//   u_j = sigma_j H' x_j - beta_{j-1} sigma_{j-1} x_{j-1}
//   alpha_j = s_j + alpha', alpha' = sigma_j u_j . x_j,
//   beta_j^2 = |u_j|^2 - alpha'^2   (= |u_j - alpha' v_j|^2 with |v_j| = 1).
// The projector dots of x_{j+1} = u_j - alpha' v_j follow from those of u_j and
// x_j in the same way.  A relative error of |x_j|^2 reaches beta_j^2 multiplied by
// (alpha'/beta_j)^2, and one of the dots those of x_{j+1} multiplied by
// |alpha'|/beta_j.  The shift keeps alpha' small beside beta_j (alpha_j settles near
// the middle of the spectrum within a few steps).  Where it does not, as with a
// V_eff of high and narrow peaks, the errors would grow from step to step: from
// alpha'^2 > beta_j^2 / 4 on, both are summed from x_{j+1} itself (kCarried), and
// below that line each step at least halves what it inherits.
// Two vector transfers per step (x_{j-1} in, x_j out; the first planes in LDS);
// 29-point cubes, 256 workgroups: 29.5 us a step (ring kernel, three transfers,
// 40.3).
// ---------------------------------------------------------------------------
constexpr double kCarried = 0.8;  // least beta_j^2 / |u_j|^2 at which sums are carried: 1 / (1 + 1/4)
struct TileLanczos {
    double al[kMaxLanczos];
    double be[kMaxLanczos];
};

template <int C>
__global__ __launch_bounds__(Tile<C>::BLOCK, 1) void lanczos_tile_kernel(LaunchArgs K) {
    using T = Tile<C>;
    constexpr int NPL = lds_planes<C>((int)sizeof(TileLanczos));
    __shared__ TileLds<C, NPL> L;
    __shared__ TileLanczos LL;
    const int tid = threadIdx.x;
    Place<C> pl;
    pl.init(tid);
    tile_begin<C>(L, tid);
    const __amdgpu_buffer_rsrc_t slr =
        make_rsrc(reinterpret_cast<double *>(K.slots) + (long long)blockIdx.x * K.slot_elems, K.slot_elems * 8);
    const long long ns = (long long)C * C * C;

    WorkSource work;
    SnapPtr Ap;
    long long qfirst, qend, qstep;
    while (work.next(K, L, tid, Ap, qfirst, qend, qstep)) {
        const auto &A = *Ap;
        const int n = A.n;
        const __amdgpu_buffer_rsrc_t vr = make_rsrc(A.veff, A.nd * 8);
        const __amdgpu_buffer_rsrc_t pr = make_rsrc(A.pgrid, A.nd * 8);
        const int kmax = (long long)A.n_lanczos < ns ? A.n_lanczos : (int)ns;
        double kw[NO + 1];
        kw[0] = 0.0;
#pragma unroll
        for (int d = 1; d <= NO; ++d) kw[d] = uniform(-0.5 * A.w[d]);
        const double kin0 = uniform(-3.0 * A.w[0]);

        for (long long q = qfirst; q < qend; q += qstep) {
            int qi, qj, qk;
            node_coords(q, n, qi, qj, qk);
            tile_setup<C>(A, L, qi, qj, qk, tid);
            const unsigned zbase = (unsigned)pmod(qk - A.m, n);
            unsigned vcol[T::NP];
            tile_columns<C>(A, pl, qi, qj, vcol);
            Vec<C> X;
            clear_prev<C, NPL>(L, tid);
            double coef[T::IPT], sx[T::IPT];  // sx: p_I . x_j
            image_coefs<C>(A, L, coef, tid);
            // adds p_I . x to L.s, x given plane by plane: f(z, v) writes a plane of the
            // thread's points
            auto projector_dots = [&](auto &&f) {
                double acc[T::NP];
#pragma unroll
                for (int r = 0; r < T::NP; ++r) acc[r] = 0.0;
#pragma unroll
                for (int z = 0; z < C; ++z) {
                    const unsigned so = (unsigned)(n * n) * ((zbase + (unsigned)z) % (unsigned)n) * 8u;
                    double x[T::NP];
                    f(z, x);
#pragma unroll
                    for (int r = 0; r < T::NP; ++r) {
                        const int i = pl.loff + z * T::LABZ + (r >> 1) * T::LW + (r & 1);
                        acc[r] += bload<double>(pr, vcol[r], so) * x[r];
                        if (acc[r] != 0.0 && (z + 1 == C || L.lab[i] != L.lab[i + T::LABZ])) {
                            atomicAdd(&L.s[L.lab[i]], acc[r]);
                            acc[r] = 0.0;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            // x_0 and its projector dots
            {
                const double *x0 = A.start + 2 * tid;
                projector_dots([&](int z, double(&x)[T::NP]) {
#pragma unroll
                    for (int r = 0; r < T::NP; ++r)
                        X.v[z][r] = x[r] = x0[(z * T::RY + (r >> 1)) * 2 * T::BLOCK + (r & 1)];
                });
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < T::IPT; ++i) {
                const int I = tid + i * T::BLOCK;
                sx[i] = I < kMaxImages ? L.s[I] : 0.0;
            }
            next_coefs<C>(L, coef, 1.0, tid);
            SweepArgs st;
            st.fa = st.fb = 0.0;
            double sig = 1.0, bprev = 0.0, gersh = 0.0;
            double shift = uniform(kin0 + A.veff[q]);
            int ksteps = kmax;
            for (int j = 0; j < kmax; ++j) {
                st.c0 = uniform(kin0 - shift);
                st.so = sig;
                st.prev = j > 0;
                double d[2] = {0.0, 0.0}, centre = 0.0;
                tile_sweep<kLanczos, C, NPL>(L, pl, X, kw, slr, vr, pr, vcol, zbase, n, st, tid, d,
                                             centre);
                tile_sum<2, C>(L, d, tid);
                const double a1 = uniform(sig * d[1]);
                double b2 = d[0] - a1 * a1;
                const double fa = uniform(a1 * sig);
                const double al = uniform(shift + a1);
                const bool direct = !(b2 > kCarried * d[0]) && j + 1 < kmax;
                if (direct) {
                    // |x_{j+1}|^2 and p_I . x_{j+1} from x_{j+1} = u_j - alpha' v_j itself
                    double e[1] = {0.0};
#pragma unroll
                    for (int i = 0; i < T::IPT; ++i) {
                        const int I = tid + i * T::BLOCK;
                        if (I < kMaxImages) L.s[I] = 0.0;
                    }
                    __syncthreads();  // every wave has read the first sums
                    projector_dots([&](int z, double(&x)[T::NP]) {
                        double pv[T::NP];
                        prev_plane<C, NPL>(L, pl, slr, z, pv, tid);
#pragma unroll
                        for (int r = 0; r < T::NP; ++r) {
                            x[r] = X.v[z][r] - fa * pv[r];
                            e[0] += x[r] * x[r];
                        }
                        pin(e[0]);
                    });
                    tile_sum<1, C>(L, e, tid);
                    b2 = e[0];
                }
                const double be = uniform(sqrt(b2 > 0.0 ? b2 : (b2 == b2 ? 0.0 : b2)));
                if (tid == 0) {
                    LL.al[j] = al;
                    LL.be[j] = be;
                    // (the last step's beta is not used)
                    if (!isfinite(al) || (j + 1 < kmax && !isfinite(be))) atomicOr(A.flags, kFlagLanczos);
                }
                gersh = fmax(gersh, fabs(al) + be + bprev);
                if (j == kmax - 1 || be <= 1e-13 * gersh) {
                    ksteps = j + 1;
                    break;
                }
                const double rb = uniform(1.0 / be);
#pragma unroll
                for (int i = 0; i < T::IPT; ++i) {
                    const int I = tid + i * T::BLOCK;
                    if (I < kMaxImages) {
                        sx[i] = direct ? L.s[I] : L.s[I] - fa * sx[i];
                        L.s[I] = 0.0;
                        L.cs[I] = rb * coef[i] * sx[i];
                    }
                }
                st.fa = fa;
                st.fb = uniform(be * sig);
                sig = rb;
                bprev = be;
                shift = al;
            }
            __syncthreads();
            if (tid < 64) sturm_extremes(ksteps, LL.al, LL.be, L.bc, tid);
            __syncthreads();
            if (tid == 0) {
                const double lmn = L.bc[0], lmx = L.bc[1];
                if (A.lmin) A.lmin[q] = lmn;
                if (A.lmax) A.lmax[q] = lmx;
                A.chi[q] = 0.5 * (lmx + lmn);
                A.zeta[q] = (1.0 + A.margin) * 0.5 * (lmx - lmn);
            }
        }
    }
}

}  // namespace

#ifdef SQ_CUBES
#define X(c)                                                                                              \
    hipError_t tile_lanczos_c##c(const LaunchArgs &a, int nwg, hipStream_t s) {                           \
        hipLaunchKernelGGL((lanczos_tile_kernel<c>), dim3(nwg), dim3(Tile<c>::BLOCK), 0, s, a);           \
        return hipGetLastError();                                                                         \
    }                                                                                                     \
    hipError_t tile_moments_c##c(const LaunchArgs &a, int nwg, hipStream_t s) {                           \
        hipLaunchKernelGGL((moments_tile_kernel<c>), dim3(nwg), dim3(Tile<c>::BLOCK), 0, s, a);           \
        return hipGetLastError();                                                                         \
    }                                                                                                     \
    hipError_t tile_occupancy_c##c(bool lanczos, int *nb) {                                               \
        const int B = Tile<c>::BLOCK;                                                                     \
        if (lanczos) return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, lanczos_tile_kernel<c>, B, 0); \
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, moments_tile_kernel<c>, B, 0);            \
    }
SQ_CUBES
#undef X
#endif

}  // namespace sq
