// steps2d.hip -- two 2D time steps per launch (eq. 3-4 with CPML, source injection, free surface,
// receiver rows and saved bands; Alg. 2 forward loop), reading level n from one buffer set and
// writing level n + 2 to the other.
//
// A workgroup owns a strip of consecutive z rows (one lane per row, 64 to 512 lanes) of one shot
// over a run of columns and marches along x, one column per iteration.  The two time steps follow
// each other as a pipeline along the march: with the newest column of p^n at k, the half steps of
// step l update v at column k - l H - N and p at column k - (l + 1) H (H = 2N - 1), so a column
// passes through four half steps while its neighbours arrive.
//   * Along x every stencil runs in registers: rings of 2N columns of p and v_x per level (the
//     loop is unrolled by 2N, so the rings are renamed, not copied).  The rings also hold the old
//     values the next step updates.
//   * Along z the stencils read one column of p or v_z per half step from LDS, written by the
//     lanes of the strip in the iteration before; two buffers each, one barrier per column.
//   * Fields are read once and written once per two steps; the loads of a column are issued D
//     iterations ahead.  The 2 H rows and columns around a workgroup's own cells are computed a
//     second time by its neighbours.
// Each cell's arithmetic is the one of the half-step kernels, so both give the same fields
// bitwise.
//
// What bounds it: the two or three wavefronts per SIMD that the rings leave room for (131 vector
// registers at order 4, about 200 at order 8).  Counted on 500 x 1500, 32 shots, boxes off: 1.6 to
// 1.8 of them resident per SIMD, an instruction in flight in 71 % of a SIMD's cycles at order 8 (48 % at
// order 4), 4.4 TB/s (4.3) of the 6.2 that a copy reaches; at order 8 62 vector instructions per cell
// and step, 37 of them on the main path of a cell, the others for halos, slabs and edges.
// Small grids wait for the serial chain of one march.  It saves launches
// (one per two steps instead of four, and instead of the source and free-surface launches beside
// them), which is what small grids and spread sources pay for, and half of the fields' traffic.
// Against the half-step kernels, 1000 steps: order 4, 500 x 1500, 1 / 4 / 16 shots 7.77 / 10.8 / 21.4
// -> 6.64 / 8.38 / 13.0 ms, 800 x 2000, 8 shots, box off 90.1 -> 66.0 ms; order 8 with off-grid
// sources, 263 x 611 below a free surface, 6 shots 19.2 -> 16.6 ms, and 4000 steps of 300 x 900,
// 16 shots 165 -> 135, 500 x 1500, 16 / 32 shots 254 / 511 -> 262 / 449 ms; order 8 on the grid it is
// between 0.86 and 1.29 of their time (500 x 1500 x 16 shots 258 -> 265 ms per 4000 steps,
// 150 x 200 x 1 shot 9.1 -> 11.7 ms), so there the half-step kernels stay the default.  Loads 4
// columns ahead instead of 2, one step per launch instead of two, and three wavefronts per SIMD at
// order 8 (by spilling) measured slower.
#include <algorithm>
#include <type_traits>

#include "smi_internal.hpp"
#include "device.hpp"
#include "side.hpp"

namespace smi {

namespace {

constexpr unsigned kOut = 0x80000000u;    // a lane offset past every buffer: reads 0, writes nothing

// sum of two lane offsets of which either, or both, may be kOut: never wraps back into the buffer
__device__ __forceinline__ unsigned add_out(unsigned a, unsigned b) {
    return __builtin_elementwise_add_sat(a, b);
}

struct SG {
    int nshot, s0;      // shots of the launch, the first of them (boxes and fields count from 0)
    int nall;           // shots of the plan (stride of the box table)
    int z0;             // first row of the first strip
    int nstrip, step;   // strips, rows between their first rows
    int nrun, R;        // runs of R columns over the widest box
    int nmain;          // workgroups of the step; the blocks after them sample receivers
    int it;             // first step of the launch
    unsigned rbytes;    // bytes from the model to the end of the receiver rows
    // receiver rows: rows [zlo, zlo + nrow) of p after every step go to the side rows [level][shot][x][row]
    int zlo, nrow;
    unsigned aside;     // their byte offset in the launch's buffer resource
    // receivers of the previous launch's levels (first step ext_it, < 0: none)
    int ext_it;
    const float *ext_side;
    float *dcal;
    unsigned *status;
};

// Saved bands (Sec. 4.2) of the levels a launch passes: slot[l] the buffer of level it + 1 + l
// (shot 0), or null.  off: offsets of the blocks (p: z faces, x faces; v_z; v_x) in a level.
struct SBand {
    float *slot[2];
    long long stride;   // floats between shots
    int pz[2], px[2], vz[2], vx[2];
};

// one receiver's sample of step it from the side rows of p after that step
__device__ __forceinline__ void side_sample(const Geom &g, const Recv &rv, const float *side, int zlo,
                                            int nrow, float *dcal, int it, unsigned *status, int r) {
    const float *sd = side + (long long)rv.shot[r] * nrow * (g.M[1] + kSidePad);
    float v = 0.f;
    for (int t = rv.toff[r]; t < rv.toff[r + 1]; ++t) {
        const int rel = (int)(rv.tcell[t] - g.org);
        const int x = rel / g.ld1, z = rel - x * g.ld1;
        v += rv.tw[t] * sd[(long long)nrow * x + z - zlo];
    }
    dcal[rv.obase[r] + (long long)it * rv.stride[r]] = v;
    if (!isfinite(v)) atomicOr(status, 2u);
}

__device__ __forceinline__ float bld(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
}
__device__ __forceinline__ void bst(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, vo, so, 0);
}

constexpr int kRows = 512;                // rows of the largest strip
constexpr int kRun = 256;                 // columns of the longest run
constexpr int kCols = kRun + 48;          // with the columns its pipeline passes
constexpr int kPad = 4;                   // LDS rows either side of a strip, always zero

// The source of a shot, kept in LDS so that it does not hold registers through the march.
template <int T>
struct Source {
    long long tw;           // weights of the source's nodes (const float *), 0: one node
    int x0, z0, nz;         // its nodes: columns from x0, rows [z0, z0 + nz)
    float scale;            // dt / dV
    float amp[T];           // source amplitude of the steps (unscaled when tw is set)
};

template <int N, int T>
struct Lds {
    // one column of p (input of step l) and of v_z (of step l), two buffers each
    float p[T][2][kRows + 2 * kPad];
    float v[T][2][kRows + 2 * kPad];
    // by column: CPML profile (a, b) along x of step l at half and integer nodes, (0, 1) where the
    // memory variable stays; byte offset of the column in the x slabs, kOut outside them
    float2 xh[T][kCols], xi[T][kCols];
    unsigned xo[kCols];
    // memory variables of d_x p and d_x v_x on their way to the next step, by column and lane
    float rx[2][2 * N][kRows];
    Source<T> src;
};

// zero, read late: keeps what is addressed through it from being loaded ahead of its branch
__device__ __forceinline__ int later() {
    int o = 0;
    asm volatile("" : "+v"(o));
    return o;
}

// one LDS word at its own immediate offset (pairs would need an address register per array)
__device__ __forceinline__ float ldsr(const float *p) { return *(const volatile __attribute__((address_space(3))) float *)(const __attribute__((address_space(3))) float *)p; }

typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) const float gcfloat;

// float at byte offset vo of a uniform address
__device__ __forceinline__ void gst(float *base, unsigned vo, float v) {
    *(gfloat *)((char *)base + vo) = v;
}

// Per-wavefront reasons to leave the main path: the source; receiver rows; saved bands of the z
// faces; saved bands of the x faces
constexpr int kEvSrc = 1, kEvRec = 2, kEvBz = 4, kEvBx = 8;

// The march of one workgroup over the columns [x0, x1) of rows [o0, o1) (its own cells), lane
// row z = zl + lane.
//   ZP: the wavefront's rows touch an absorbing slab along z.
//   XE: the run's columns (with their halo) reach past the computing box of a step or into an
//       absorbing slab along x; otherwise no column needs a check.
// The pipeline fills in blocks of U columns: block b runs the first b of the 2T half steps, the
// columns after them run all and store, a multiple of U of them (columns past the box keep their
// value, so storing them changes nothing).
template <int N, int T, int D, bool ZP, bool XE, bool FS, bool SAVE>
__device__ __forceinline__ void march(const Geom &g, const Fields &A, const Fields &B,
                                      const Model &m, const Cpml &cp, const int *__restrict__ box,
                                      const SG &sg, const SBand &sb, Lds<N, T> &lds, int s, int zl,
                                      int o0, int o1, int x0, int x1, int ev, int sx0, int sxw) {
    constexpr int U = 2 * N, H = 2 * N - 1, M = U - 1;
    static_assert(T == 2 && U % D == 0, "two steps; the load ring divides the unrolled block");
    const int lane = (int)threadIdx.x;
    const int z = zl + lane;
    const long long so = (long long)s * g.P;
    const unsigned colb = 4u * (unsigned)g.ld1;
    // one buffer resource over the model, both field sets and the receiver rows; byte offsets of
    // the arrays in it (the second field set has the layout of the first)
    const char *rb = (const char *)m.kdt;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(rb), (short)0, (int)sg.rbytes, 0x00020000);
    auto off = [&](const float *p) { return (unsigned)((const char *)p - rb); };
    const unsigned abz = off(m.bdt[0]), abx = off(m.bdt[1]);
    const unsigned ap = off(A.p + so), avz = off(A.v[0] + so), avx = off(A.v[1] + so);
    const unsigned aqz = off(A.psp[0] + s * g.psz[0]), auz = off(A.psv[0] + s * g.psz[0]);
    const unsigned aqx = off(A.psp[1] + s * g.psz[1]), aux = off(A.psv[1] + s * g.psz[1]);
    const unsigned dst = off(B.p) - off(A.p);
    // Cells outside the computing box of a step take no update: there the coefficients read as 0
    // (lane offset kOut) and the memory variables keep their value (profile a = 0, b = 1).
    bool zin[T];
    unsigned vm[T];
    int xlo[T];
    unsigned xw[T];
    const unsigned vr = z < g.M[0] ? 4u * (unsigned)(z + GH) : kOut;
#pragma unroll
    for (int l = 0; l < T; ++l) {
        const int *b = box + ((long long)l * sg.nall + s) * 6;
        zin[l] = z >= b[0] && z < b[1];
        vm[l] = zin[l] ? vr : kOut;
        xlo[l] = b[2];
        xw[l] = (unsigned)(b[3] - b[2]);
    }
    const bool own = z >= o0 && z < o1;
    const int zr = z - g.nb;                        // row counted from a free surface
    const unsigned vw = own && zin[T - 1] ? vr : kOut;
    // CPML along z
    int zs = -1;
    float zah[T], zbh[T], zai[T], zbi[T];
    if (ZP) {
        zs = z >= 0 && z < g.M[0] ? slab_index(z, g.M[0], g.nb) : -1;
#pragma unroll
        for (int l = 0; l < T; ++l) {
            const bool in = zs >= 0 && zin[l];
            zah[l] = in ? cp.a_h[0][z] : 0.f;
            zbh[l] = in ? cp.b_h[0][z] : 1.f;
            zai[l] = in ? cp.a_i[0][z] : 0.f;
            zbi[l] = in ? cp.b_i[0][z] : 1.f;
        }
    }
    const unsigned vq = zs >= 0 ? 4u * (unsigned)zs : kOut;
    const unsigned vqw = own && zin[T - 1] ? vq : kOut;
    const unsigned vxq = z >= 0 && z < g.M[0] ? 4u * (unsigned)z : kOut;
    const unsigned vxw = own && zin[T - 1] ? vxq : kOut;
    const unsigned wzb = 4u * (unsigned)g.W;
    // lane offsets of the receiver rows (with a free surface, also of the image rows this lane
    // holds) and of the z faces of a saved level
    unsigned vsd = kOut, vsm = kOut, vpb = kOut, vvb = kOut;
    if (own) {
        const int rr = z - sg.zlo;
        const bool img = FS && zr < 0 && zr >= -N;
        if ((unsigned)rr < (unsigned)sg.nrow && !img) vsd = 4u * (unsigned)rr;
        if (FS && zr > 0 && zr <= N && (unsigned)(rr - 2 * zr) < (unsigned)sg.nrow) vsm = 4u * (unsigned)(rr - 2 * zr);
        if (SAVE) {
            const int n0 = g.n[0];
            const int p0 = FS ? N - zr : zr + N, v0 = FS ? N - 1 - zr : zr + N;
            if ((unsigned)p0 < (unsigned)N) vpb = 4u * (unsigned)(sb.pz[0] + p0);
            if ((unsigned)(zr - n0) < (unsigned)N) vpb = 4u * (unsigned)(sb.pz[1] + zr - n0);
            if ((unsigned)v0 < (unsigned)N) vvb = 4u * (unsigned)(sb.vz[0] + v0);
            if ((unsigned)(zr - n0 + 1) < (unsigned)N) vvb = 4u * (unsigned)(sb.vz[1] + zr - n0 + 1);
        }
    }
    const float psgn = FS && zr <= N ? -1.f : 1.f;   // the image rows of p are odd
    const unsigned sdc = 4u * (unsigned)sg.nrow;
    const unsigned asd = sg.aside + (unsigned)s * sdc * (unsigned)(g.M[1] + kSidePad);
    const unsigned sdl = (unsigned)sg.nall * sdc * (unsigned)(g.M[1] + kSidePad);

    float pw[T][U], vx[T][U], vz[T][U];     // rings by column
    float qz[U], uz[U];                     // memory variables of d_z p, d_z v_z on their way to the next step
#pragma unroll
    for (int j = 0; j < U; ++j) {
        qz[j] = uz[j] = 0.f;
#pragma unroll
        for (int l = 0; l < T; ++l) pw[l][j] = vx[l][j] = vz[l][j] = 0.f;
    }
    struct Ld {         // loads in flight of one iteration
        float p, vx, vz, bx[T], bz[T], kd[T], qz, uz, qx, ux;
    };
    Ld q[D];
    const int ks = x0 + T * H - 2 * T * U;          // first column
    auto colo = [&](int c) { return colb * (unsigned)((XE ? max(c, -GH) : c) + GH); };
    auto gcol = [&](int c) { return (unsigned)(XE ? min(max(c, 0), g.M[1] - 1) : c); };
    // Columns of p and v past the shot's frame read its last column, which is always zero: the next
    // shot's field lies there, and what it holds need not be finite.  (At order 4 what a stored
    // column depends on, T H and at most U - 1 columns past the grid, stays within the two frames.)
    constexpr bool kPast = T * H + U - 1 > 2 * GH;
    auto colf = [&](int c) { return colo(XE && kPast ? min(c, g.M[1] + GH - 1) : c); };
    auto load = [&](int k, Ld &L) __attribute__((always_inline)) {
        L.p = bld(rs, vr, ap + colf(k));
        const unsigned cv = colf(k - N);
        L.vx = bld(rs, vr, avx + cv);
        L.vz = bld(rs, vr, avz + cv);
#pragma unroll
        for (int l = 0; l < T; ++l) {
            const int c = k - l * H - N, e = k - (l + 1) * H;
            const unsigned vc = !XE || (unsigned)(c - xlo[l]) < xw[l] ? vm[l] : kOut;
            const unsigned ve = !XE || (unsigned)(e - xlo[l]) < xw[l] ? vm[l] : kOut;
            L.bx[l] = bld(rs, vc, abx + colo(c));
            L.bz[l] = bld(rs, vc, abz + colo(c));
            L.kd[l] = bld(rs, ve, colo(e));
        }
        if (ZP) {
            L.qz = bld(rs, vq, aqz + wzb * gcol(k - N));
            L.uz = bld(rs, vq, auz + wzb * gcol(k - H));
        }
        if (XE) {
            L.qx = bld(rs, add_out(vxq, lds.xo[k - N - ks]), aqx);
            L.ux = bld(rs, add_out(vxq, lds.xo[k - H - ks]), aux);
        }
    };
    // what the source adds to this lane's p of step l at column c
    auto source = [&](int l, int c) __attribute__((always_inline)) {
        const Source<T> *sd = &lds.src + later();
        const int tz = z - sd->z0;
        float a = 0.f;
        if ((unsigned)tz < (unsigned)sd->nz) {
            gcfloat *tw = (gcfloat *)sd->tw;
            a = tw ? src_amp(src_amp(sd->scale, tw[(c - sd->x0) * sd->nz + tz]), sd->amp[l]) : sd->amp[l];
        }
        return a;
    };
    // one block of U columns from kb on, with the first ACT half steps running
    auto block = [&](auto act, int kb) __attribute__((always_inline)) {
        constexpr int ACT = decltype(act)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int k = __builtin_amdgcn_readfirstlane(kb + u);
            asm volatile("" : "+s"(k));     // keeps each column's offsets and compares from being hoisted
            const int par = u & 1;
            const Ld c = q[u % D];
            load(k + D, q[u % D]);
            pw[0][u] = c.p;
            // the rows around this one that the z-stencils of the iteration read
            float zp[T][2 * N], zv[T][2 * N];
#pragma unroll
            for (int l = 0; l < T; ++l)
#pragma unroll
                for (int d = 0; d < 2 * N; ++d) {
                    if (ACT > 2 * l && d != N - 1) zp[l][d] = ldsr(&lds.p[l][par][lane + kPad + d - (N - 1)]);
                    if (ACT > 2 * l + 1 && (FS || d != N)) zv[l][d] = ldsr(&lds.v[l][par][lane + kPad + d - N]);
                }
            float2 ah[T], ai[T];
            if (XE)
#pragma unroll
                for (int l = 0; l < T; ++l) {
                    if (ACT > 2 * l) ah[l] = lds.xh[l][k - l * H - N - ks];
                    if (ACT > 2 * l + 1) ai[l] = lds.xi[l][k - (l + 1) * H - ks];
                }
            float pt = 0.f;                 // p after the last step
#pragma unroll
            for (int l = 0; l < T; ++l) {
                if (ACT > 2 * l) {
                    // v_z, v_x of step l at column cv
                    const int cv = k - l * H - N;
                    const int sv = (u + 4 * U - l * H - N) & M;
                    float ez = 0.f, ex = 0.f;
#pragma unroll
                    for (int d = 1; d <= N; ++d) {
                        ez += g.c[0][d - 1] * (zp[l][N - 1 + d] - (d == 1 ? pw[l][sv] : zp[l][N - d]));
                        ex += g.c[1][d - 1] * (pw[l][(sv + d) & M] - pw[l][(sv + U + 1 - d) & M]);
                    }
                    if (ZP) {
                        const float nz = __builtin_fmaf(zbh[l], l == 0 ? c.qz : qz[sv], zah[l] * ez);
                        if (l + 1 < T) qz[sv] = nz;
                        else bst(rs, (ACT < 2 * T && cv < x0) || (XE && cv >= g.M[1]) ? kOut : vqw,
                                 aqz + dst + wzb * (unsigned)cv, nz);
                        ez += nz;
                    }
                    if (XE) {
                        const float nx = __builtin_fmaf(ah[l].y, l == 0 ? c.qx : ldsr(&lds.rx[0][sv][lane]), ah[l].x * ex);
                        if (l + 1 < T) lds.rx[0][sv][lane] = nx;
                        else bst(rs, ACT < 2 * T && cv < x0 ? kOut : add_out(vxw, lds.xo[cv - ks]), aqx + dst, nx);
                        ex += nx;
                    }
                    vz[l][sv] = (l == 0 ? c.vz : vz[l ? l - 1 : 0][sv]) - c.bz[l] * ez;
                    vx[l][sv] = (l == 0 ? c.vx : vx[l ? l - 1 : 0][sv]) - c.bx[l] * ex;
                }
                if (ACT > 2 * l + 1) {
                    // p of step l at column cq
                    const int cq = k - (l + 1) * H;
                    const int sp = (u + 4 * U - (l + 1) * H) & M;
                    float ez = 0.f, ex = 0.f;
#pragma unroll
                    for (int d = 1; d <= N; ++d) {
                        ez += g.c[0][d - 1] * ((!FS && d == 1 ? vz[l][sp] : zv[l][N + d - 1]) - zv[l][N - d]);
                        ex += g.c[1][d - 1] * (vx[l][(sp + d - 1) & M] - vx[l][(sp + U - d) & M]);
                    }
                    if (ZP) {
                        const float nz = __builtin_fmaf(zbi[l], l == 0 ? c.uz : uz[sp], zai[l] * ez);
                        if (l + 1 < T) uz[sp] = nz;
                        else bst(rs, XE && cq >= g.M[1] ? kOut : vqw, auz + dst + wzb * (unsigned)cq, nz);
                        ez += nz;
                    }
                    if (XE) {
                        const float nx = __builtin_fmaf(ai[l].y, l == 0 ? c.ux : ldsr(&lds.rx[1][sp][lane]), ai[l].x * ex);
                        if (l + 1 < T) lds.rx[1][sp][lane] = nx;
                        else bst(rs, add_out(vxw, lds.xo[cq - ks]), aux + dst, nx);
                        ex += nx;
                    }
                    float sdiv = 0.f;
                    sdiv += ez;
                    sdiv += ex;
                    float pn = pw[l][sp] - c.kd[l] * sdiv;
                    if (__builtin_expect((ev & kEvSrc) && (unsigned)(cq - sx0) <= (unsigned)sxw, 0)) {
                        const float a = source(l, cq);
                        // (as p + amplitude, on the rows of the source alone)
                        if (a != 0.f) pn += a;
                    }
                    if (FS) pn = zr == 0 ? 0.f : pn;
                    if (l + 1 < T) pw[l + 1 < T ? l + 1 : 0][sp] = pn;
                    else pt = pn;
                }
            }
            if (ACT == 2 * T) {
                const int c = k - T * H;
                const int sc = (u + 4 * U - T * H) & M;
                const unsigned co = dst + colo(c);
                const float vzs = vz[T - 1][sc];
                bst(rs, vw, avx + co, vx[T - 1][sc]);
                if (FS) {
                    // free surface: v_z even and p odd about it, the image rows above it written
                    // by the lanes of the rows they mirror
                    const unsigned vf = zr >= 0 || zr < -N ? vw : kOut;
                    bst(rs, vf, avz + co, vzs);
                    bst(rs, vf, ap + co, pt);
                    if (zr >= 0 && zr < N) bst(rs, vw - 4u * (unsigned)(1 + 2 * zr), avz + co, vzs);
                    if (zr > 0 && zr <= N) bst(rs, vw - 8u * (unsigned)zr, ap + co, -pt);
                } else {
                    bst(rs, vw, avz + co, vzs);
                    bst(rs, vw, ap + co, pt);
                }
            }
            if (ACT > 2 && __builtin_expect(ev & (kEvRec | kEvBz | kEvBx), 0)) {
#pragma unroll
                for (int l = 0; l < T; ++l) {
                    if (l > 0 && ACT < 2 * T) continue;
                    const int c = k - (l + 1) * H;
                    const int sc = (u + 4 * U - (l + 1) * H) & M;
                    if (ACT < 2 * T && c < x0) continue;
                    const float pn = l + 1 < T ? pw[l + 1 < T ? l + 1 : 0][sc] : pt;
                    if (ev & kEvRec) {
                        // Columns past the run's own hold what the next run stores there, or zeros
                        // past the box: a last run is rounded up to U columns, and the first level
                        // is H columns ahead of the last.  The rows have room for them (a test of
                        // the column costs 1 % of a small launch).
                        static_assert((T - 1) * H + U - 1 <= kSidePad, "receiver rows too short");
                        const unsigned co = asd + l * sdl + sdc * (unsigned)c;
                        bst(rs, vsd, co, pn);
                        if (FS) bst(rs, vsm, co, -pn);
                    }
                    if (SAVE && (ev & (kEvBz | kEvBx)) && sb.slot[l] && c < x1) {
                        const int xi = c - g.nb, n0 = g.n[0], n1 = g.n[1];
                        float *b = sb.slot[l] + s * sb.stride;
                        if ((ev & kEvBz) && (unsigned)xi < (unsigned)n1) {
                            const unsigned co = 4u * N * (unsigned)xi;
                            if (vpb != kOut) gst(b, vpb + co, FS ? psgn * pn : pn);
                            if (vvb != kOut) gst(b, vvb + co, vz[l][sc]);
                        }
                        if ((ev & kEvBx) && ((unsigned)(xi + N) < (unsigned)N || xi >= n1 - 1)) {
                            if (own && (unsigned)zr < (unsigned)n0) {
                                const int e0 = xi + N, e1 = xi - n1, f1 = xi - n1 + 1;
                                if ((unsigned)e0 < (unsigned)N) {
                                    gst(b, 4u * (unsigned)(sb.px[0] + zr + n0 * e0), pn);
                                    gst(b, 4u * (unsigned)(sb.vx[0] + zr + n0 * e0), vx[l][sc]);
                                }
                                if ((unsigned)e1 < (unsigned)N) gst(b, 4u * (unsigned)(sb.px[1] + zr + n0 * e1), pn);
                                if ((unsigned)f1 < (unsigned)N) gst(b, 4u * (unsigned)(sb.vx[1] + zr + n0 * f1), vx[l][sc]);
                            }
                        }
                    }
                }
            }
            // the columns the next iteration's z-stencils read
#pragma unroll
            for (int l = 0; l < T; ++l) {
                const float pl = pw[l][(u + 4 * U - l * H - N + 1) & M];
                const float vl = vz[l][(u + 4 * U - (l + 1) * H + 1) & M];
                float *P = &lds.p[l][par ^ 1][lane + kPad], *V = &lds.v[l][par ^ 1][lane + kPad];
                if (l == 0 || ACT > 2 * l - 1) {
                    if (FS && l > 0) {
                        if (zr >= 0 || zr < -N) *P = pl;
                        if (zr > 0 && zr <= N && lane >= 2 * zr) P[-2 * zr] = -pl;
                    } else {
                        *P = pl;
                    }
                }
                if (ACT > 2 * l) {
                    if (FS) {
                        if (zr >= 0 || zr < -N) *V = vl;
                        if (zr >= 0 && zr < N && lane >= 1 + 2 * zr) V[-1 - 2 * zr] = vl;
                    } else {
                        *V = vl;
                    }
                }
            }
            __syncthreads();
        }
    };
    // block 0: the first U columns of p alone
#pragma unroll
    for (int u = 0; u < U; ++u) pw[0][u] = bld(rs, vr, ap + colo(ks + u));
#pragma unroll
    for (int j = 0; j < D; ++j) load(ks + U + j, q[j]);
    lds.p[0][0][lane + kPad] = pw[0][U - N];
    __syncthreads();
    block(std::integral_constant<int, 1>{}, ks + U);
    block(std::integral_constant<int, 2>{}, ks + 2 * U);
    block(std::integral_constant<int, 3>{}, ks + 3 * U);
    for (int kb = ks + 2 * T * U; kb - T * H < x1; kb += U) block(std::integral_constant<int, 2 * T>{}, kb);
}

template <int N, int T, int D, bool FS, bool SAVE>
__global__ __launch_bounds__(kRows) void k_steps2d(Geom g, Fields A, Fields B, Model m, Cpml cp,
                                                   const int *__restrict__ box, SG sg, SBand sb,
                                                   Recv rv, const long long *__restrict__ src_cell,
                                                   const int *__restrict__ toff,
                                                   const long long *__restrict__ tcell,
                                                   const float *__restrict__ tw,
                                                   const float *__restrict__ stf, int nt) {
    constexpr int H = 2 * N - 1;
    __shared__ Lds<N, T> lds;
    const int nl = (int)blockDim.x;
    const int sidel = sg.nall * sg.nrow * (g.M[1] + kSidePad);
    if ((int)blockIdx.x >= sg.nmain) {
        // receivers of the previous launch's levels, from its side rows
        const int nthr = ((int)gridDim.x - sg.nmain) * nl;
        for (int q = ((int)blockIdx.x - sg.nmain) * nl + (int)threadIdx.x; q < T * rv.R; q += nthr) {
            const int l = q / rv.R, r = q - l * rv.R;
            if (sg.ext_it + l < nt)
                side_sample(g, rv, sg.ext_side + (long long)l * sidel, sg.zlo, sg.nrow, sg.dcal,
                            sg.ext_it + l, sg.status, r);
        }
        return;
    }
    // strip fastest, then run, then shot, in XCD-contiguous ranges: neighbouring workgroups
    // share their overlapping rows and columns in one L2
    const int L = xcd_remap((int)blockIdx.x, sg.nmain);
    const int strip = L % sg.nstrip;
    int r = L / sg.nstrip;
    const int run = r % sg.nrun;
    const int s = sg.s0 + r / sg.nrun;
    const int *b = box + ((long long)(T - 1) * sg.nall + s) * 6;
    const int zl = sg.z0 + strip * sg.step;
    const int o0 = strip == 0 ? -GH : zl + T * H;
    const int o1 = strip + 1 == sg.nstrip ? g.M[0] : zl + sg.step + T * H;
    const int x0 = b[2] + run * sg.R, x1 = min(x0 + sg.R, b[3]);
    if (x0 >= x1 || o1 <= b[0] || o0 >= b[1]) return;
    // zero rows either side of the strip, and both buffers of every column
    for (int i = (int)threadIdx.x; i < T * 4 * (kRows + 2 * kPad); i += nl) (&lds.p[0][0][0])[i] = 0.f;
    const int *bl = box + (long long)s * 6;     // the boxes of the steps, nall * 6 apart
    {
        const int c0 = x0 + T * H - 4 * T * N;
        for (int i = (int)threadIdx.x; i < kCols; i += nl) {
            const int c = c0 + i;
            const int xs = c >= 0 && c < g.M[1] ? slab_index(c, g.M[1], g.nb) : -1;
            lds.xo[i] = xs >= 0 ? 4u * (unsigned)g.ld1 * (unsigned)xs : kOut;
#pragma unroll
            for (int l = 0; l < T; ++l) {
                const int *q = bl + (long long)l * sg.nall * 6;
                const bool in = xs >= 0 && c >= q[2] && c < q[3];
                lds.xh[l][i] = in ? make_float2(cp.a_h[1][c], cp.b_h[1][c]) : make_float2(0.f, 1.f);
                lds.xi[l][i] = in ? make_float2(cp.a_i[1][c], cp.b_i[1][c]) : make_float2(0.f, 1.f);
            }
        }
    }
    // the source's nodes: one (src_cell >= 0), or the block between its first and last node
    const int t0 = toff[s], t1 = toff[s + 1];
    const int c0 = (int)(tcell[t0] - g.org), c1 = (int)(tcell[t1 - 1] - g.org);
    const int sx0 = c0 / g.ld1, sz0 = c0 - sx0 * g.ld1;
    const int sx1 = c1 / g.ld1, sz1 = c1 - sx1 * g.ld1;
    if (threadIdx.x == 0) {
        Source<T> &d = lds.src;
        const bool one = src_cell[s] >= 0;
        d.tw = one ? 0 : (long long)(tw + t0);
        d.scale = g.src_scale;
        d.x0 = sx0;
        d.z0 = sz0;
        d.nz = sz1 - sz0 + 1;
#pragma unroll
        for (int l = 0; l < T; ++l) {
            const float a = sg.it + l < nt ? stf[(long long)s * nt + sg.it + l] : 0.f;
            d.amp[l] = one ? src_amp(g.src_scale, a) : a;
        }
    }
    __syncthreads();
    const int w0 = zl + ((int)threadIdx.x & ~63), w1 = w0 + 64;     // the wavefront's rows
    int ev = 0;
    if (sz0 < w1 && sz1 >= w0 && sx0 < x1 + T * H && sx1 >= x0 - T * H && sg.it < nt) ev |= kEvSrc;
    if (sg.zlo < w1 && sg.zlo + sg.nrow + (FS ? 2 * N : 0) > w0) ev |= kEvRec;
    if (SAVE) {
        if ((w0 < g.nb + N + 1 && w1 > g.nb - N) || w1 > g.nb + g.n[0] - 1) ev |= kEvBz;
        if (x0 < g.nb + N || x1 > g.nb + g.n[1] - 1) ev |= kEvBx;
    }
    ev = __builtin_amdgcn_readfirstlane(ev);
    const bool zp = w0 < g.nb || w1 > g.M[0] - g.nb - 1;
    const bool xe = x0 - T * H < max(bl[2], g.nb) || x1 + T * H > min(bl[3], g.M[1] - g.nb - 1);
    auto go = [&](auto zpt, auto xet) __attribute__((always_inline)) {
        march<N, T, D, decltype(zpt)::value, decltype(xet)::value, FS, SAVE>(
            g, A, B, m, cp, box, sg, sb, lds, s, zl, o0, o1, x0, x1, ev, sx0, sx1 - sx0);
    };
    const std::true_type yes{};
    const std::false_type no{};
    if (xe) {
        if (__builtin_amdgcn_readfirstlane((int)zp)) go(yes, yes);
        else go(no, yes);
    } else {
        if (__builtin_amdgcn_readfirstlane((int)zp)) go(yes, no);
        else go(no, no);
    }
}

// strips of 64 w lanes over the rows [z0, z1) with h halo rows per side: their number, and the
// rows between their first rows (a multiple of 32: every strip starts on a storage line)
int strips_of(int w, int rows, int h, int &step) {
    step = (64 * w - 2 * h) / 32 * 32;
    if (64 * w >= rows) return 1;
    return step > 0 ? 1 + (rows - 64 * w + step - 1) / step : 0;
}

template <int N>
hipError_t steps_t(const StepCtx &c, const Fields &src, const Fields &dst, int it, int par) {
    constexpr int T = kSteps, H = 2 * N - 1, D = 2;
    const Plan &pl = *c.pl;
    const Views &w = *c.w;
    if (!pl.side || it < 0 || it + T > pl.nrun) return hipErrorInvalidValue;   // no rows, or no boxes
    const int s0 = c.s0, s1 = shot_end(c);
    int z0 = pl.M[0], z1 = 0, ex = 0;
    for (int s = s0; s < s1; ++s) {
        const int *b = &pl.fbox[((size_t)(it + T - 1) * pl.nshot + s) * 6];
        z0 = std::min(z0, b[0]);
        z1 = std::max(z1, b[1]);
        ex = std::max(ex, b[3] - b[2]);
    }
    // (the image rows that rows of the box read are written by lanes of their own)
    if (pl.g.freesurf && z0 < pl.g.nb + N) z0 = std::min(z0, pl.g.nb - N);
    z0 = zalign(z0);
    const int rows = z1 - z0;
    // Strip height (64 W lanes) and run length: the least modelled time over the rounds in which
    // the workgroups run.  A CU holds 12 wavefronts of the order-4 kernel (8 of order 8) and, by its
    // LDS, 3 workgroups (2), a run of R columns takes R + 8 T iterations, and an iteration gets
    // slower with the wavefronts that share a SIMD (about 0.3 of its time alone for each further one).
    constexpr int kWaves = N == 2 ? 12 : 8, kGroups = 160 * 1024 / (int)sizeof(Lds<N, T>);
    int W = kRows / 64, nstrip = 1, step = 0, R = 2 * N;
    double best = 0;
    for (int q = kRows / 64; q >= 1; --q) {
        int st = 0;
        const int n = strips_of(q, rows, T * H, st);
        if (n <= 0) continue;
        const int cap = std::max(1, std::min(kWaves / q, kGroups));     // workgroups resident on a CU
        for (int r = 2 * N; r <= kRun; r += r < 64 ? 2 * N : 16) {
            const long long nwg = (long long)(s1 - s0) * n * ((ex + r - 1) / r);
            const long long rounds = (nwg + 256 * cap - 1) / (256 * cap);
            const int res = (int)std::min<long long>(cap, (nwg + 255) / 256);
            const double cost = (double)rounds * (r + 8 * T) * (1.0 + 0.3 * std::max(0.0, res * q / 4.0 - 1.0));
            if (best == 0 || cost < best) {
                best = cost;
                W = q;
                nstrip = n;
                step = st;
                R = r;
            }
        }
    }
    SG sg{};
    sg.nshot = s1 - s0;
    sg.s0 = s0;
    sg.nall = pl.nshot;
    sg.z0 = z0;
    sg.nstrip = nstrip;
    sg.step = step;
    sg.R = R;
    sg.nrun = (ex + R - 1) / R;
    sg.nmain = sg.nshot * nstrip * sg.nrun;
    sg.it = it;
    sg.rbytes = (unsigned)(pl.off_side + side_bytes(pl) - pl.off_model);
    sg.zlo = pl.rec_zlo;
    sg.nrow = pl.rec_nrow;
    const size_t half = side_bytes(pl) / 8;
    sg.aside = (unsigned)(pl.off_side - pl.off_model + 4 * par * half);
    Recv rv = w.recv;
    const int r0 = pl.rec_off[s0], r1 = pl.rec_off[s1];
    rv.R = r1 - r0;
    rv.shot += r0;
    rv.obase += r0;
    rv.stride += r0;
    rv.toff += r0;
    sg.ext_it = c.ext_it;
    sg.ext_side = w.side + (par ^ 1) * half;
    sg.dcal = c.ext_dcal;
    sg.status = w.status;
    int extra = 0;
    if (c.ext_it >= 0 && rv.R > 0) extra = std::min(256, (T * rv.R + 64 * W - 1) / (64 * W));
    SBand sb{};
    const int dr = pl.g.dr;
    if (pl.save) {
        sb.stride = (long long)pl.nsave * pl.band.B;
        for (int l = 0; l < T; ++l) {
            const int lev = it + 1 + l;
            if (lev % dr == 0 && lev / dr < pl.nsave) sb.slot[l] = w.bands + (size_t)(lev / dr) * pl.band.B;
        }
        for (int k = 0; k < 2; ++k) {       // block order of the plan: p left, right, v left, right
            sb.pz[k] = (int)pl.band.blk[k].off;
            sb.vz[k] = (int)pl.band.blk[2 + k].off;
            sb.px[k] = (int)pl.band.blk[4 + k].off;
            sb.vx[k] = (int)pl.band.blk[6 + k].off;
        }
    }
    const int *box = w.fbox + (size_t)it * pl.nshot * 6;
    const dim3 grid((unsigned)(sg.nmain + extra)), block(64u * (unsigned)W);
    auto launch = [&](auto fs, auto sv) -> hipError_t {
        constexpr bool F = decltype(fs)::value, V = decltype(sv)::value;
        hipLaunchKernelGGL((k_steps2d<N, T, D, F, V>), grid, block, 0, c.st, pl.geom, src, dst,
                           w.model, w.cpml, box, sg, sb, rv, (const long long *)w.src_cell,
                               (const int *)w.src_toff, (const long long *)w.src_tcell,
                               (const float *)w.src_tw, c.stf, pl.g.nt);
        return hipGetLastError();
    };
    const std::true_type yes{};
    const std::false_type no{};
    if (pl.g.freesurf) return pl.save ? launch(yes, yes) : launch(yes, no);
    if constexpr (N == 2)
        if (pl.save) return launch(no, yes);
    return pl.save ? hipErrorInvalidValue : launch(no, no);     // (see steps2d_available)
}

// receivers of the levels of one launch (first step it) from its side rows
__global__ __launch_bounds__(256) void k_side_extract(Geom g, Recv rv, const float *side, int sidel,
                                                      int zlo, int nrow, float *dcal, int it, int nl,
                                                      unsigned *status) {
    const int q = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (q >= nl * rv.R) return;
    const int l = q / rv.R;
    side_sample(g, rv, side + (long long)l * sidel, zlo, nrow, dcal, it + l, status, q - l * rv.R);
}

}  // namespace

bool steps2d_available(const Plan &pl) {
    if (pl.nd != 2 || !pl.dbuf || !pl.side) return false;
    // with a free surface a lane holds at most one row of the saved z faces
    if (pl.g.freesurf && pl.n[0] <= pl.N + 1) return false;
    // order 8 saving bands without a free surface: the slower one nearly everywhere (see below), not
    // compiled
    if (pl.N == 4 && pl.save && !pl.g.freesurf) return false;
    // 31-bit byte offsets from the model over both field sets and the receiver rows
    return pl.off_side + side_bytes(pl) - pl.off_model < (size_t(1) << 31) - (1u << 20);
}

// Where they are the default.  Time of a forward pass against the half-step kernels' (two cells per
// lane where those are small): geometric mean and range over 40 x 40 to 500 x 1500 cells, 1 to 32
// shots, boxes on and off.  A source that spreads over several nodes costs the half-step kernels a
// launch per step, two below a free surface; saving bands takes the marching loop's wavefronts at the
// faces off their main path and spills its scalar registers.
//   without saved bands: order 4 0.81 (0.61-0.95), below a free surface 0.87 (0.65-1.02), spread
//     sources 0.65 (0.54-0.83), both 0.51 (0.39-0.74); order 8 with spread sources below a free
//     surface 0.92 (0.75-1.10), without one 0.98 (0.78-1.16), but 1.21 (1.08-1.29) on less than
//     32768 padded cells per shot; order 8 with sources on the grid 0.86 to 1.29
//   with them: order 4 1.01 (0.75-1.21), every fifth level 0.95 (0.69-1.10), spread sources 0.77
//     (0.61-1.07), also below a free surface 0.72 (0.54-1.45), there with sources on the grid 1.23
//     (0.87-1.90); order 8 with spread sources 1.31 (1.03-1.62), every fifth level 1.17
//     (0.91-1.46), below a free surface 1.06 (0.93-1.48), every fifth level there 0.99 (0.87-1.32)
bool steps2d_default(const Plan &pl) {
    if (!steps2d_available(pl)) return false;
    if (pl.N == 2) return !pl.save || pl.src_multi || !pl.g.freesurf;
    if (!pl.src_multi) return false;
    if (pl.g.freesurf) return !pl.save || pl.g.dr > 1;
    return (long long)pl.M[0] * pl.M[1] >= 32768;
}

hipError_t fwd_steps_2d(const StepCtx &c, const Fields &src, const Fields &dst, int it, int par) {
    return c.pl->N == 2 ? steps_t<2>(c, src, dst, it, par) : steps_t<4>(c, src, dst, it, par);
}

hipError_t steps2d_extract(const StepCtx &c, int it, int par, float *dcal) {
    const Plan &pl = *c.pl;
    const Views &w = *c.w;
    Recv rv = w.recv;
    const int r0 = pl.rec_off[c.s0], r1 = pl.rec_off[shot_end(c)];
    rv.R = r1 - r0;
    rv.shot += r0;
    rv.obase += r0;
    rv.stride += r0;
    rv.toff += r0;
    const int nl = std::min(kSteps, pl.g.nt - it);
    if (rv.R == 0 || nl <= 0) return hipSuccess;
    const int sidel = (int)(side_bytes(pl) / (8 * kSteps));
    hipLaunchKernelGGL(k_side_extract, dim3((unsigned)((nl * rv.R + 255) / 256)), dim3(256), 0, c.st,
                       pl.geom, rv, (const float *)(w.side + side_bytes(pl) / 8 * par), sidel,
                       pl.rec_zlo, pl.rec_nrow, dcal, it, nl, w.status);
    return hipGetLastError();
}

}  // namespace smi
