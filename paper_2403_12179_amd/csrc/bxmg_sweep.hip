// Streaming smoother: two red-black sweeps of a one-box level in one pass over
// its data, with the residual that follows them or the prolongation before
// them; the coefficient constant, or in FP32 a cell beta or face arrays.
//
// One half-sweep per launch moves 1.5 arrays per half-sweep, 6 for the two
// sweeps of a V(2,2) cycle and 2 more for the residual after them.  Here a
// block owns a column of the domain (XM pairs x TY rows x ZC planes) and
// walks it in z, plane by plane; each thread holds one x-pair (2m, 2m+1) of
// one row.  At the step that loads plane q, the four half-sweeps and the
// residual work on the planes behind it:
//
//   stage 1  colour 0 of plane q-1      stage 3  colour 0 of plane q-3
//   stage 2  colour 1 of plane q-2      stage 4  colour 1 of plane q-4
//   stage 5  the residual of plane q-5
//
// Every stage's z neighbours and own cells are in the thread's registers
// (its column's last few planes); of its x and y neighbours one is the
// thread's own other cell and three come from LDS, written there one step
// earlier by the stage before (one barrier per step).  So f and one colour of
// u are read once (the other's old values only beside Dirichlet faces, where a
// ghost holds them) and u written once.  A block recomputes a halo around its own columns
// (one layer per stage), reading u of one array and writing another: blocks
// need nothing of each other.  The arithmetic of a cell, and the order of
// its sums, are those of the one-colour kernel, so the results are bitwise
// those of one launch per half-sweep: a ghost beyond a Dirichlet face holds
// minus the cell's own value before the update (reading own registers), and
// periodic columns wrap.
//
// A block's wait for ghosts and its selects between a ghost and a cell are
// compiled for the walls it touches (none, an x face alone, any).
//
// Measured on the 256^3 FP64 Dirichlet level 0: two sweeps, residual and
// restriction 160 us, against 4 x 50 + 66 us one launch each; two sweeps after
// the coarse levels with the interpolation and the norms 217, against 58 + 4 x
// 50 + 66.  The arrays alone (352 MB: half of u, f, u out, an eighth for the
// coarse level) take 75 us at the 4.67 TB/s of a large copy; loads, stores,
// LDS traffic (18 to 26 reads and 6 writes of a value per thread and step) and
// FP64 issue (85 to 110 instructions) overlap only in part, as a block's waves
// run the same phase of a step together.  The 256^3 solve went from 8.78 to
// 5.57 ms, the 192^3 heat step from 4.49 to 2.61 ms.  Adding an FP32
// correction to the FP64 iterate (kSweepAdd) takes 455 us over the 52 million
// cells of 64 problems, 250 of which are its bytes at the copy rate.
//
// With a coefficient (FP32) a thread has the 9 faces of its pair formed once
// per plane and kept in 60 registers: a half-sweep launch forms 6 harmonic
// means per cell, each a division.  Bound by that arithmetic (about 240
// instructions a step, 140 of them the 13 divisions) times the recomputed
// halo: 512^3, cell beta, sweeps from zero with residual and restriction 1380
// us against 4 x 396 + 615, sweeps after the coarse levels 1255 against 256 + 4
// x 396; 256^3 with face arrays 160 and 180 us against 4 x 60 + 97 and 85 + 4 x
// 60.  With the direction pass below and the fused coarse cycle the 512^3
// preconditioned solve went from 158 to 113 ms and the 128^3 mixed one from 6.7
// to 5.2 (both versions in turn on one card).  In FP64 the same form takes 340
// registers a thread before and 298 after the coarse levels: one wave a SIMD
// in blocks of 256 threads, and 205 spilled in blocks of 512.  It is not built.
#include <hip/hip_runtime.h>
#include <type_traits>

#include <algorithm>
#include <vector>

#include "bxmg_device.h"

namespace bxmg {

// KIND (SweepKind): what follows the sweeps.  ZERO: they start from u = 0,
// which is not read.  POST: the sweeps after the coarse levels, whose
// correction (ec, the next level's u) is interpolated on the way in: colour 1
// as it enters, colour 0's old value only where it is read, beside Dirichlet
// faces.  The coarse planes of a block's columns go through LDS, four at a
// time, a ghost there being the cell it mirrors (minus, beyond a Dirichlet
// face); a thread carries one value of the next plane.  So the prolongation
// costs 8 LDS reads a pair and no pass of its own: 256^3 FP64, sweeps and norms
// 217 us with it, 197 without, and 58 the three launches that it took; 192^3
// 87 against 85 + 34.
// No ghost is read or written.
// NT: threads per block (columns of a block, halo included, at most NT).
// kSweepAdd: the result is added to acc (and its face ghosts refreshed)
// instead of being stored.  JOBS: many levels in one launch; block b works
// block where[b].y of job where[b].x (none: -1).
// MODE: 0 constant coefficient; 1 cell beta, faces are harmonic means; 2 face
// arrays (fat).  The coefficients of a pair's faces and their sums are formed
// (or loaded) once per plane, for all stages, and stay in registers.
template <class T, int NT, bool ZERO, int KIND, bool POST, bool JOBS, int MODE>
__global__ void __launch_bounds__(NT) k_sweep(SweepArgs A0, const SweepArgs* __restrict__ jobs,
                                             const int2* __restrict__ where, const T* __restrict__ uin,
                                             T* __restrict__ uout, const T* __restrict__ f, T* __restrict__ cf,
                                             double* __restrict__ acc, double* __restrict__ partials,
                                             const int* __restrict__ active, const T* __restrict__ beta,
                                             const FaceArrays<T>* __restrict__ fat, const T* __restrict__ ec) {
    using std::integral_constant;
    constexpr bool REST = KIND == kSweepRestrict, NORM = KIND == kSweepNorm, ADD = KIND == kSweepAdd;
    constexpr bool RES = REST || NORM;
    // LDS half planes (one colour of one plane of the block's columns)
    constexpr int bB0 = 0, bR1 = 2, bB2 = 4, bR3 = 6, bB4 = 10, bS = 12, bK = REST ? 14 : RES ? 12 : 10;
    constexpr int bC = bK + (MODE == 1 ? 4 : 0);  // (bK, bK + 2: beta of colour 0, 1)
    __shared__ T lds[(bC + (POST ? 4 : 0)) * NT];  // bC: coarse planes
    const int tid = threadIdx.x;
    // block -> (bx, by, bz), neighbouring blocks on one XCD
    int blk = blockIdx.x, job = 0;
    if constexpr (JOBS) {
        job = where[blk].x;
        blk = where[blk].y;
        if (job < 0) return;
    } else {
        const int nb = gridDim.x;
        if ((nb & 7) == 0) blk = (blk & 7) * (nb >> 3) + (blk >> 3);
    }
    const SweepArgs A = JOBS ? jobs[job] : A0;
    if (active && !active[A.pid]) return;
    if constexpr (JOBS) {
        uin += A.uin;
        uout += A.uout;
        f += A.f;
        cf += A.cf;
        acc += A.acc;
        ec += A.ec;
    }
    const int bx = blk % A.nbx, byz = blk / A.nbx;
    const int by = byz % A.nby, bz = byz / A.nby;
    const int nm = A.n[0] >> 1, n1 = A.n[1], n2 = A.n[2];
    const int ty = tid / A.RM, tm = tid - ty * A.RM;
    // the thread's column: pair m of row y (raw: before periodic wrapping)
    const int mr = bx * A.XM - A.hm + tm, yr = by * A.TY - A.hy + ty;
    int m = mr, y = yr;
    bool in = ty < A.RY;
    if (A.per[0]) { m %= nm; m += m < 0 ? nm : 0; } else in = in && m >= 0 && m < nm;
    if (A.per[1]) { y %= n1; y += y < 0 ? n1 : 0; } else in = in && y >= 0 && y < n1;
    const bool own = in && tm >= A.hm && tm < A.hm + A.XM && mr < nm && ty >= A.hy && ty < A.hy + A.TY && yr < n1;
    const bool perz = A.per[2] != 0;
    // Dirichlet faces the column lies on
    const bool fxl = in && !A.per[0] && m == 0, fxr = in && !A.per[0] && m == nm - 1;
    const bool fyl = in && !A.per[1] && y == 0, fyr = in && !A.per[1] && y == n1 - 1;
    const bool edge_y = __ballot(fyl || fyr) != 0, edge_xy = edge_y || __ballot(fxl || fxr) != 0;
    const int z0 = bz * A.ZC, zlim = min(z0 + A.ZC, n2);
    // first plane loaded: the halo below, rounded to an even plane so that a
    // step's plane parity is known at compile time
    constexpr int kHalo = (RES ? 5 : 4) - (ZERO && MODE != 1 ? 1 : 0), kFirst = (kHalo + 1) & ~1;
    const int zs = perz ? z0 - kFirst : max(0, z0 - kFirst);
    const int zend = zlim + (REST ? 6 : RES ? 5 : 4);  // one past the last step
    const int zmax = min(zlim + (RES ? 4 : 3), perz ? zlim + 4 : n2 - 1);  // last plane with values in use
    // cells of the pair: in a plane of parity p, the colour-c cell is at
    // x = 2m + o, o = (c + y + p) & 1; "A" offsets belong to o = yo, "B" ones
    // to o = 1 - yo
    const int yo = y & 1;
    // LDS slots of the x neighbours of the pair's cells and of the rows beside
    // (a neighbour outside the block's columns is never used by an own cell)
    const bool wx = A.per[0] && A.hm == 0, wy = A.per[1] && A.hy == 0;
    const int sl = tm > 0 ? tid - 1 : wx ? tid + A.RM - 1 : tid;
    const int sr = tm < A.RM - 1 ? tid + 1 : wx ? tid - (A.RM - 1) : tid;
    const int sdn = !in ? tid : ty > 0 ? tid - A.RM : wy ? tid + (A.RY - 1) * A.RM : tid;
    const int sup = !in ? tid : ty < A.RY - 1 ? tid + A.RM : wy ? tid - (A.RY - 1) * A.RM : tid;
    const int sxA = !in ? tid : yo ? sr : sl;
    const int sxB = !in ? tid : yo ? sl : sr;
    // the pair's cell on a Dirichlet x face, if any
    const bool fxA = yo ? fxr : fxl, fxB = yo ? fxl : fxr;
    const int es = (int)sizeof(T);
    const int row = (y + 1) * A.H + m, co = A.cs * es, pl = A.GH * es;
    const int vA = in ? (row + yo) * es : kOffPastBox, vB = in ? (row + 1 - yo) * es : kOffPastBox;
    // POST: the block's coarse columns, one per thread (its offset in a plane,
    // parity and sign), and the pair's place among them
    const int y0 = by * A.TY - A.hy, cy0 = (y0 >> 1) - 1, CW = A.RM + 2;
    int ci = 0, cp = 0, ic = 0;
    bool cin = false, cneg = false;
    if constexpr (POST) {
        const int cy = tid / CW, nr = ((y0 + A.RY - 1) >> 1) + 2 - cy0;
        cin = cy < nr;
        auto mirror = [&](int v, int n, int per) {
            if (per) {
                v %= n;
                return v < 0 ? v + n : v;
            }
            const bool out = v < 0 || v >= n;
            cneg = cneg != out;
            v = v < 0 ? -1 - v : v >= n ? 2 * n - 1 - v : v;
            return min(max(v, 0), n - 1);  // (columns further out are never used)
        };
        const int I = mirror(bx * A.XM - A.hm - 1 + tid - cy * CW, nm, A.per[0]);
        const int J = mirror(cy0 + cy, n1 >> 1, A.per[1]);
        ci = cin ? ((J + 1) * A.cH + ((I + 1) >> 1)) * (int)sizeof(T) : kOffPastBox;
        cp = (I + J + A.cpar) & 1;
        ic = in ? ((yr >> 1) - cy0) * CW + tm + 1 : CW + 1;
    }
    const T h2 = uniform((T)(A.h * A.h)), ih2 = uniform((T)(1.0 / (A.h * A.h)));
    const T dg = uniform((T)(A.a * (A.h * A.h))), sb = uniform(T(6) + dg);
    Recip<T> rsb(sb);
    rsb.b = sb;
    rsb.yh = uniform(rsb.yh);
    rsb.yl = uniform(rsb.yl);
    const int bytes = 2 * A.cs * es;
    const auto Ru = __builtin_amdgcn_make_buffer_rsrc((void*)(ZERO ? f : uin), (short)0, bytes, kBufferDword3);
    const auto Rf = __builtin_amdgcn_make_buffer_rsrc((void*)f, (short)0, bytes, kBufferDword3);
    const auto Ro = __builtin_amdgcn_make_buffer_rsrc((void*)uout, (short)0, bytes, kBufferDword3);
    const auto Rc = __builtin_amdgcn_make_buffer_rsrc((void*)(POST ? ec : f), (short)0,
                                                      POST ? 2 * A.ccs * es : bytes, kBufferDword3);
    // kSweepAdd: the same cells of acc, loaded with the plane four ahead (a
    // load after a step's stores would wait for them)
    const auto Ra = __builtin_amdgcn_make_buffer_rsrc((void*)(ADD ? (const void*)acc : (const void*)f), (short)0,
                                                      2 * A.cs * 8, kBufferDword3);
    const int aA = own ? (row + yo) * 8 : kOffPastBox, aB = own ? (row + 1 - yo) * 8 : kOffPastBox;
    double a0[4] = {}, a1[4] = {};  // indexed by plane modulo 4

    // MODE 1: the cell beta; MODE 2: the face arrays and the pair's offsets in
    // them (x: the outer faces of the A and B cell; y, z: the cell's lower face)
    const auto Rk = __builtin_amdgcn_make_buffer_rsrc((void*)(MODE == 1 ? beta : f), (short)0, bytes, kBufferDword3);
    __amdgpu_buffer_rsrc_t R0, R1, R2;
    int ox = 0, oxA = 0, oxB = 0, oyA = 0, oyB = 0, ozA = 0, ozB = 0, px = 0, py = 0, pz = 0;
    if constexpr (MODE == 2) {
        const FaceArrays<T> fa = fat[A.pid];
        const int n0 = A.n[0];
        px = (n0 + 1) * n1 * es;
        py = n0 * (n1 + 1) * es;
        pz = n0 * n1 * es;
        R0 = __builtin_amdgcn_make_buffer_rsrc((void*)fa.c[0], (short)0, px * n2, kBufferDword3);
        R1 = __builtin_amdgcn_make_buffer_rsrc((void*)fa.c[1], (short)0, py * n2, kBufferDword3);
        R2 = __builtin_amdgcn_make_buffer_rsrc((void*)fa.c[2], (short)0, pz * (n2 + 1), kBufferDword3);
        const int xr = 2 * m + (n0 + 1) * y, yr0 = 2 * m + n0 * y;
        ox = in ? (xr + 1) * es : kOffPastBox;
        oxA = in ? (xr + 2 * yo) * es : kOffPastBox;
        oxB = in ? (xr + 2 - 2 * yo) * es : kOffPastBox;
        oyA = ozA = in ? (yr0 + yo) * es : kOffPastBox;
        oyB = ozB = in ? (yr0 + 1 - yo) * es : kOffPastBox;
    }

    // the column's registers, indexed by plane modulo 8 (only a few of each
    // are live): values of colour 0 (r) and 1 (b) after 0..4 half-sweeps
    T r0[8], b0[8], r1[8], b2[8], r3[8], b4[8], fr[8], fb[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        r0[k] = T(0); b0[k] = T(0); r1[k] = T(0); b2[k] = T(0);
        r3[k] = T(0); b4[k] = T(0); fr[k] = T(0); fb[k] = T(0);
    }
    // coefficients of the colour-c cell: inner (shared) and outer x face, y
    // faces, lower z face, the sum of its faces; be: MODE 1's cell beta
    T kin[8], ko[2][8], kd[2][8], ku[2][8], zl[2][8], ks[2][8], be[2][8];
    if constexpr (MODE != 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            kin[k] = T(0);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                ko[c][k] = T(0); kd[c][k] = T(0); ku[c][k] = T(0);
                zl[c][k] = T(0); ks[c][k] = T(0); be[c][k] = T(0);
            }
        }
    }
    T sprev = T(0), half = T(0);  // restriction: this row's pair sum, the even plane's sum of four
    double mx = 0.0, s2 = 0.0;
    int nbad = 0;  // non-finite residuals

    // loads of plane q into ring slot PH (plane parity PH & 1)
    auto load = [&](auto ph, int q) {
        constexpr int PH = decltype(ph)::value;
        int z = min(q, zmax);  // planes past the last one in use: any values
        if (perz) {            // (twice: the halo may be wider than the domain)
            z += z < 0 ? n2 : 0;
            z += z < 0 ? n2 : 0;
            z -= z >= n2 ? n2 : 0;
            z -= z >= n2 ? n2 : 0;
        }
        const int zo = (z + 1) * pl;
        const int vr = (PH & 1) ? vB : vA, vb = (PH & 1) ? vA : vB;
        fr[PH] = Raw<T>::ld(Rf, vr, zo);
        fb[PH] = Raw<T>::ld(Rf, vb, zo + co);
        if constexpr (MODE == 1) {
            be[0][PH] = Raw<T>::ld(Rk, vr, zo);
            be[1][PH] = Raw<T>::ld(Rk, vb, zo + co);
        }
        if constexpr (MODE == 2) {
            kin[PH] = Raw<T>::ld(R0, ox, z * px);
            ko[0][PH] = Raw<T>::ld(R0, (PH & 1) ? oxB : oxA, z * px);
            ko[1][PH] = Raw<T>::ld(R0, (PH & 1) ? oxA : oxB, z * px);
            const int yr = (PH & 1) ? oyB : oyA, yb = (PH & 1) ? oyA : oyB, row1 = A.n[0] * es;
            kd[0][PH] = Raw<T>::ld(R1, yr, z * py);
            ku[0][PH] = Raw<T>::ld(R1, yr, z * py + row1);
            kd[1][PH] = Raw<T>::ld(R1, yb, z * py);
            ku[1][PH] = Raw<T>::ld(R1, yb, z * py + row1);
            // (past a Dirichlet domain: the face on its upper side)
            const int zf = !perz && q == n2 ? n2 : z;
            zl[0][PH] = Raw<T>::ld(R2, (PH & 1) ? ozB : ozA, zf * pz);
            zl[1][PH] = Raw<T>::ld(R2, (PH & 1) ? ozA : ozB, zf * pz);
        }
        if constexpr (ADD) {
            const bool mine = q - 4 >= z0 && q - 4 < zlim;
            const int zd = mine ? (q - 3) * A.GH * 8 : 0;
            a0[PH & 3] = Raw<double>::ld(Ra, !mine ? kOffPastBox : (PH & 1) ? aB : aA, zd);
            a1[PH & 3] = Raw<double>::ld(Ra, !mine ? kOffPastBox : (PH & 1) ? aA : aB, zd + A.cs * 8);
        }
        if constexpr (!ZERO) {
            b0[PH] = Raw<T>::ld(Ru, vb, zo + co);
            // colour 0's old value is read only through Dirichlet ghosts
            r0[PH] = T(0);  // (or each slot's last value would stay live)
            if (edge_xy || (!perz && (z == 0 || z == n2 - 1))) r0[PH] = Raw<T>::ld(Ru, vr, zo);
        }
    };
    // coarse plane K of the block (wrapped or mirrored; its sign: cneg and beyond)
    T cr = T(0);
    auto load_coarse = [&](int K) {
        const int nk = n2 >> 1;
        const int below = perz ? K + nk : -1 - K, above = perz ? K - nk : 2 * nk - 1 - K;
        K = K < 0 ? below : K >= nk ? above : K;
        if (perz) K = K < 0 ? K + nk : K >= nk ? K - nk : K;  // (twice, as above)
        K = min(max(K, 0), nk - 1);
        return Raw<T>::ld(Rc, ci + ((cp + K) & 1) * (A.ccs * es), (K + 1) * A.cGH * es);
    };
    auto put_coarse = [&](int slot, int K, T v) {
        const bool beyond = !perz && (K < 0 || K >= (n2 >> 1));
        if (cin) lds[(bC + slot) * NT + tid] = cneg != beyond ? -v : v;
    };

    // EDGE: 0 inside, 1 beside a Dirichlet x face, 2 beside any
    auto step = [&](auto ph, auto edge, int q) {
        constexpr int PH = decltype(ph)::value, EDGE = decltype(edge)::value;
#define RS(d) ((PH - (d) + 16) & 7)   /* ring slot of plane q - d */
#define ISA(d, c) ((((c) + PH - (d)) & 1) == 0)  /* its colour-c cell is at o = yo */
        struct Three { T x, d, u; };
        auto near = [&](int buf, bool isA) {
            const T* hp = lds + buf * NT;
            return Three{hp[isA ? sxA : sxB], hp[sdn], hp[sup]};
        };
        // neighbour sum of the colour-c cell of plane q - D: own_o = the
        // pair's other cell; oldv = the cell's own value before the update
        // (x- + x+ commutes, so the own cell's side does not matter)
        auto sum = [&](auto dd, auto cc, bool isA, T own_o, Three n, T zm, T zp, T oldv) {
            constexpr int D = decltype(dd)::value, C = decltype(cc)::value;
            if constexpr (EDGE > 0) {
                const T g = -oldv;
                n.x = (isA ? fxA : fxB) ? g : n.x;
                if constexpr (EDGE > 1) {
                    n.d = fyl ? g : n.d;
                    n.u = fyr ? g : n.u;
                    zm = !perz && q == D ? g : zm;
                    zp = !perz && q == D + n2 - 1 ? g : zp;
                }
            }
            if constexpr (MODE == 0) return ((own_o + n.x) + (n.d + n.u)) + (zm + zp);
            else
                return ((kin[RS(D)] * own_o + ko[C][RS(D)] * n.x) + (kd[C][RS(D)] * n.d + ku[C][RS(D)] * n.u)) +
                       (zl[C][RS(D)] * zm + zl[1 - C][RS(D - 1)] * zp);
        };
        // the cell's new value from (neighbour sum - h^2 f)
        auto relax = [&](auto dd, auto cc, T v) {
            if constexpr (MODE == 0) return rsb.div(v);
            else return v / ks[decltype(cc)::value][RS(decltype(dd)::value)];
        };
        constexpr integral_constant<int, 0> c0{};
        constexpr integral_constant<int, 1> c1{};
        if constexpr (POST) {
            // the correction at the colour-c cell of plane q: its parent and the
            // neighbours towards it
            auto interp = [&](int c) {
                constexpr int kr = PH >> 1;  // coarse plane modulo 4, from the first
                const T* a = lds + (bC + (kr & 3)) * NT + ic;
                const T* b = lds + (bC + (((PH & 1) ? kr + 1 : kr + 3) & 3)) * NT + ic;
                const int dx = ISA(0, c) == (yo != 0) ? 1 : -1, dyc = yo ? CW : -CW;
                const T c000 = a[0], c100 = a[dx], c010 = a[dyc], c001 = b[0];
                const T c110 = a[dx + dyc], c101 = b[dx], c011 = b[dyc], c111 = b[dx + dyc];
                const T v =
                    (((T(27) * c000 + T(9) * ((c100 + c010) + c001)) + T(3) * ((c110 + c101) + c011)) + c111) *
                    T(0.015625);
                return A.order == 1 ? c000 : v;
            };
            b0[RS(0)] = b0[RS(0)] + interp(1);
            if constexpr (EDGE > 0) r0[RS(0)] = r0[RS(0)] + interp(0);
            if constexpr ((PH & 1) == 0) {
                put_coarse(((PH >> 1) + 1) & 3, (q >> 1) + 1, cr);
                cr = load_coarse((q >> 1) + 2);
            }
            if constexpr (NORM || MODE != 0) __builtin_amdgcn_sched_barrier(0);
        }
        // every LDS value of the step, written in earlier steps (in parts where
        // all of them at once would spill)
        constexpr bool kTight = POST && (NORM || MODE != 0);
        Three t1{}, t2, t3, t4, t5r{}, t5b{};
        T spart = T(0);
        if constexpr (!ZERO) t1 = near(bB0 + ((PH - 1) & 1), ISA(1, 0));
        t2 = near(bR1 + ((PH - 1) & 1), ISA(2, 1));
        auto near34 = [&] {
            t3 = near(bB2 + ((PH - 1) & 1), ISA(3, 0));
            t4 = near(bR3 + ((PH - 1) & 3), ISA(4, 1));
        };
        if constexpr (!kTight) near34();
        auto near5 = [&] {
            t5r = near(bB4 + ((PH - 1) & 1), ISA(5, 0));
            t5b = near(bR3 + ((PH - 2) & 3), ISA(5, 1));
        };
        if constexpr (RES && !kTight) near5();
        if constexpr (REST) spart = lds[(bS + ((PH - 1) & 1)) * NT + sup];
        if constexpr (MODE == 1) {
            const Three k0 = near(bK + 2 + ((PH - 1) & 1), ISA(1, 0)), k1 = near(bK + ((PH - 1) & 1), ISA(1, 1));
            lds[(bK + (PH & 1)) * NT + tid] = be[0][RS(0)];
            lds[(bK + 2 + (PH & 1)) * NT + tid] = be[1][RS(0)];
            kin[RS(1)] = harm(be[0][RS(1)], be[1][RS(1)]);
            // beyond a Dirichlet face beta is the cell's own
            auto faces = [&](auto cc, bool isA, Three k) {
                constexpr int C = decltype(cc)::value;
                T lo = be[1 - C][RS(1)], hi = be[C][RS(0)];
                if constexpr (EDGE > 0) {
                    const T b = be[C][RS(1)];
                    k.x = (isA ? fxA : fxB) ? b : k.x;
                    if constexpr (EDGE > 1) {
                        k.d = fyl ? b : k.d;
                        k.u = fyr ? b : k.u;
                        lo = !perz && q == 0 ? hi : lo;
                        hi = !perz && q == n2 ? lo : hi;
                    }
                }
                ko[C][RS(1)] = harm(be[C][RS(1)], k.x);
                kd[C][RS(1)] = harm(k.d, be[C][RS(1)]);
                ku[C][RS(1)] = harm(be[C][RS(1)], k.u);
                zl[C][RS(0)] = harm(lo, hi);
            };
            faces(c0, ISA(1, 0), k0);
            faces(c1, ISA(1, 1), k1);
        }
        if constexpr (MODE != 0) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
                ks[c][RS(1)] = (((kin[RS(1)] + ko[c][RS(1)]) + (kd[c][RS(1)] + ku[c][RS(1)])) +
                                (zl[c][RS(1)] + zl[1 - c][RS(0)])) + dg;
        }
        // plane q enters: colour 1 for stage 1's neighbours
        if constexpr (!ZERO) lds[(bB0 + (PH & 1)) * NT + tid] = b0[RS(0)];
        {  // stage 1
            T su = T(0);
            if constexpr (!ZERO)
                su = sum(integral_constant<int, 1>(), c0, ISA(1, 0), b0[RS(1)], t1, b0[RS(2)], b0[RS(0)], r0[RS(1)]);
            r1[RS(1)] = relax(integral_constant<int, 1>(), c0, su - h2 * fr[RS(1)]);
            lds[(bR1 + (PH & 1)) * NT + tid] = r1[RS(1)];
        }
        {  // stage 2
            const T su = sum(integral_constant<int, 2>(), c1, ISA(2, 1), r1[RS(2)], t2, r1[RS(3)], r1[RS(1)],
                             ZERO ? T(0) : b0[RS(2)]);
            b2[RS(2)] = relax(integral_constant<int, 2>(), c1, su - h2 * fb[RS(2)]);
            lds[(bB2 + (PH & 1)) * NT + tid] = b2[RS(2)];
        }
        if constexpr (kTight) {
            __builtin_amdgcn_sched_barrier(0);
            near34();
        }
        {  // stage 3
            const T su = sum(integral_constant<int, 3>(), c0, ISA(3, 0), b2[RS(3)], t3, b2[RS(4)], b2[RS(2)], r1[RS(3)]);
            r3[RS(3)] = relax(integral_constant<int, 3>(), c0, su - h2 * fr[RS(3)]);
            lds[(bR3 + (PH & 3)) * NT + tid] = r3[RS(3)];
        }
        {  // stage 4
            const T su = sum(integral_constant<int, 4>(), c1, ISA(4, 1), r3[RS(4)], t4, r3[RS(5)], r3[RS(3)], b2[RS(4)]);
            b4[RS(4)] = relax(integral_constant<int, 4>(), c1, su - h2 * fb[RS(4)]);
            if constexpr (RES) lds[(bB4 + (PH & 1)) * NT + tid] = b4[RS(4)];
        }
        {  // plane q-4 is final
            const int p = q - 4;
            const bool mine = p >= z0 && p < zlim;
            const int zo = mine ? (p + 1) * pl : 0;  // (see kOffPastBox)
            const int vr = (PH & 1) ? vB : vA, vb = (PH & 1) ? vA : vB;
            if constexpr (!ADD) {  // (stores past the box are dropped)
                Raw<T>::st(Ro, own && mine ? vr : kOffPastBox, zo, r3[RS(4)]);
                Raw<T>::st(Ro, own && mine ? vb : kOffPastBox, zo + co, b4[RS(4)]);
            } else {
                const int cd = A.cs * 8, zd = mine ? (p + 1) * A.GH * 8 : 0;
                const double x0 = a0[PH & 3] + (double)r3[RS(4)], x1 = a1[PH & 3] + (double)b4[RS(4)];
                const int ar = (PH & 1) ? aB : aA, ab = (PH & 1) ? aA : aB;
                Raw<double>::st(Ra, mine ? ar : kOffPastBox, zd, x0);
                Raw<double>::st(Ra, mine ? ab : kOffPastBox, zd + cd, x1);
                // the face ghosts that mirror the cells
                const bool fz = p == 0 || p == n2 - 1;
                if (mine && own && (fz || m == 0 || m == nm - 1 || y == 0 || y == n1 - 1)) {
                    const int rb = (y + 1) * A.H, pd = A.GH * 8;
                    auto ghost = [&](bool per, double v, int c, int image, int below, int zi, int zb) {
                        // the periodic image (same colour) or the ghost beyond (the other colour)
                        if (per) Raw<double>::st(Ra, image * 8, zi + (c ? cd : 0), v);
                        else Raw<double>::st(Ra, below * 8, zb + (c ? 0 : cd), -v);
                    };
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const double v = c ? x1 : x0;
                        const int o = (c + y + PH) & 1, xs = m + o;  // slot of x = 2m + o in its row
                        if (m == 0 && o == 0) ghost(A.per[0], v, c, rb + nm, rb, zd, zd);
                        if (m == nm - 1 && o == 1) ghost(A.per[0], v, c, rb, rb + nm, zd, zd);
                        if (y == 0) ghost(A.per[1], v, c, (n1 + 1) * A.H + xs, xs, zd, zd);
                        if (y == n1 - 1) ghost(A.per[1], v, c, xs, (n1 + 1) * A.H + xs, zd, zd);
                        if (p == 0) ghost(perz, v, c, rb + xs, rb + xs, (n2 + 1) * pd, 0);
                        if (p == n2 - 1) ghost(perz, v, c, rb + xs, rb + xs, 0, (n2 + 1) * pd);
                    }
                }
            }
        }
        if constexpr (RES) {  // stage 5
            if constexpr (kTight) {
                __builtin_amdgcn_sched_barrier(0);
                near5();
            }
            const T sur =
                sum(integral_constant<int, 5>(), c0, ISA(5, 0), b4[RS(5)], t5r, b4[RS(6)], b4[RS(4)], r3[RS(5)]);
            const T rr = fr[RS(5)] - (sur - (MODE == 0 ? sb : ks[0][RS(5)]) * r3[RS(5)]) * ih2;
            const T sub =
                sum(integral_constant<int, 5>(), c1, ISA(5, 1), r3[RS(5)], t5b, r3[RS(6)], r3[RS(4)], b4[RS(5)]);
            const T rb = fb[RS(5)] - (sub - (MODE == 0 ? sb : ks[1][RS(5)]) * b4[RS(5)]) * ih2;
            if constexpr (NORM) {
                const int p = q - 5;
                const bool mine = own && p >= z0 && p < zlim;
#pragma unroll
                for (int c = 0; c < 2; ++c) {  // acc_norm, without branches: 0 adds nothing
                    const double v = mine ? (double)(c ? rb : rr) : 0.0, a = fabs(v);
                    const bool fine = a <= 1.7976931348623157e308;
                    mx = fmax(mx, fine ? a : 0.0);
                    nbad += fine ? 0 : 1;
                    s2 = s2 + v * v;
                }
            } else {
                // the four residuals of this row pair in plane q-6 (the
                // partner's sum arrived with the last barrier), then this
                // row's sum for the next step
                const T four = sprev + spart;
                if constexpr (((PH - 6) & 1) == 0) {
                    half = four;
                } else {
                    const int p = q - 6;
                    if (own && !(y & 1) && p >= z0 && p < zlim) {
                        const int J = y >> 1, K = p >> 1;
                        const int c = (m + J + K + A.cpar) & 1;
                        cf[(long long)c * A.ccs + (long long)(K + 1) * A.cGH + (J + 1) * A.cH + ((m + 1) >> 1)] =
                            (half + four) * T(0.125);
                    }
                }
                sprev = rr + rb;  // even x + odd x: which colour is which commutes
                lds[(bS + (PH & 1)) * NT + tid] = sprev;
            }
        }
#undef RS
#undef ISA
    };

    if constexpr (POST) {
        const T a = load_coarse((zs >> 1) - 1), b = load_coarse(zs >> 1);
        cr = load_coarse((zs >> 1) + 1);
        put_coarse(3, (zs >> 1) - 1, a);
        put_coarse(0, zs >> 1, b);
        lds_barrier();
    }
    load(integral_constant<int, 0>(), zs);
    load(integral_constant<int, 1>(), zs + 1);
    for (int qb = zs;; qb += 8) {
#define BXMG_STEP(PH)                                                                          \
    {                                                                                          \
        const int q = qb + PH;                                                                 \
        if (q >= zend) break;                                                                  \
        load(integral_constant<int, (PH + 2) & 7>(), q + 2);                                   \
        if (edge_y || (!perz && (q <= 5 || q >= n2 - 1)))                                      \
            step(integral_constant<int, PH>(), integral_constant<int, 2>(), q);                \
        else if (edge_xy) step(integral_constant<int, PH>(), integral_constant<int, 1>(), q);  \
        else step(integral_constant<int, PH>(), integral_constant<int, 0>(), q);               \
        lds_barrier();                                                                         \
    }
        BXMG_STEP(0) BXMG_STEP(1) BXMG_STEP(2) BXMG_STEP(3)
        BXMG_STEP(4) BXMG_STEP(5) BXMG_STEP(6) BXMG_STEP(7)
#undef BXMG_STEP
    }
    if constexpr (NORM) {
        double* sh = (double*)lds;  // every LDS read ended with the last barrier
        double bad = (double)nbad;
        block_reduce3(mx, s2, bad, sh);
        if (tid == 0) {
            partials[3 * (size_t)blk] = mx;
            partials[3 * (size_t)blk + 1] = s2;
            partials[3 * (size_t)blk + 2] = bad;
        }
    }
}

// One conjugate-gradient direction on a one-box level in one pass:
//   p' = (double) e + beta p,  q = L p',  partial sums of p'.q.
// A block walks a column in z as k_sweep does, p' of a plane formed as it
// enters and q one plane behind it; each face coefficient of a pair is formed
// once (MODE 1: the cell beta; 0: constant).  p and pn differ; ghosts are not
// read (minus the own cell beyond a Dirichlet face, own beta there) nor
// written.  Same operations per cell as k_kr_axpy and k_kr_apply.
// Bound by its bytes (36 a cell with e in FP32) and, with MODE 1, by 9 FP64
// divisions a pair: 512^3, FP32 e, MODE 1 1180 us, 1030 of them its bytes at the
// copy rate; the two launches took 715 + 1415, the second with 12 divisions a
// pair and 6 more FP64 loads a cell.
constexpr int kDirThreads = 512;
template <class E, int MODE>
__global__ void __launch_bounds__(kDirThreads, 4)
    k_kr_direction(SweepArgs A, const E* __restrict__ e, const double* __restrict__ p, double* __restrict__ pn,
                   const double* __restrict__ beta, double* __restrict__ q_, const KrylovScalars* __restrict__ sc,
                   double* __restrict__ partials, const int* __restrict__ active) {
    using std::integral_constant;
    constexpr int NT = kDirThreads, bP = 0, bK = 4;  // + 2 colour + plane parity
    __shared__ double lds[(MODE ? 8 : 4) * NT];
    if (active && !active[A.pid]) return;
    const double bs = sc->beta;
    const int tid = threadIdx.x;
    int blk = blockIdx.x;
    {
        const int nb = gridDim.x;
        if ((nb & 7) == 0) blk = (blk & 7) * (nb >> 3) + (blk >> 3);
    }
    const int bx = blk % A.nbx, byz = blk / A.nbx;
    const int by = byz % A.nby, bz = byz / A.nby;
    const int nm = A.n[0] >> 1, n1 = A.n[1], n2 = A.n[2];
    const int ty = tid / A.RM, tm = tid - ty * A.RM;
    const int mr = bx * A.XM - A.hm + tm, yr = by * A.TY - A.hy + ty;
    int m = mr, y = yr;
    bool in = ty < A.RY;
    if (A.per[0]) { m %= nm; m += m < 0 ? nm : 0; } else in = in && m >= 0 && m < nm;
    if (A.per[1]) { y %= n1; y += y < 0 ? n1 : 0; } else in = in && y >= 0 && y < n1;
    const bool own = in && tm >= A.hm && tm < A.hm + A.XM && mr < nm && ty >= A.hy && ty < A.hy + A.TY && yr < n1;
    const bool perz = A.per[2] != 0;
    const bool fxl = in && !A.per[0] && m == 0, fxr = in && !A.per[0] && m == nm - 1;
    const bool fyl = in && !A.per[1] && y == 0, fyr = in && !A.per[1] && y == n1 - 1;
    const int z0 = bz * A.ZC, zlim = min(z0 + A.ZC, n2);
    const int zs = perz ? z0 - 2 : max(0, z0 - 2), zend = zlim + 1;
    const int zmax = perz ? zlim : min(zlim, n2 - 1);
    const int yo = y & 1;
    const bool wx = A.per[0] && A.hm == 0, wy = A.per[1] && A.hy == 0;
    const int sl = tm > 0 ? tid - 1 : wx ? tid + A.RM - 1 : tid;
    const int sr = tm < A.RM - 1 ? tid + 1 : wx ? tid - (A.RM - 1) : tid;
    const int sdn = !in ? tid : ty > 0 ? tid - A.RM : wy ? tid + (A.RY - 1) * A.RM : tid;
    const int sup = !in ? tid : ty < A.RY - 1 ? tid + A.RM : wy ? tid - (A.RY - 1) * A.RM : tid;
    const int sxA = !in ? tid : yo ? sr : sl;
    const int sxB = !in ? tid : yo ? sl : sr;
    const bool fxA = yo ? fxr : fxl, fxB = yo ? fxl : fxr;
    constexpr int es = (int)sizeof(E);
    const int row = (y + 1) * A.H + m;
    const int oA = in ? row + yo : -1, oB = in ? row + 1 - yo : -1;
    const int vA = in ? oA * 8 : kOffPastBox, vB = in ? oB * 8 : kOffPastBox;
    const int eA = in ? oA * es : kOffPastBox, eB = in ? oB * es : kOffPastBox;
    const int wA = own ? vA : kOffPastBox, wB = own ? vB : kOffPastBox;
    const int co = A.cs * 8, pl = A.GH * 8;
    const double ih2 = 1.0 / (A.h * A.h), dg = A.a * (A.h * A.h);
    const auto Re = __builtin_amdgcn_make_buffer_rsrc((void*)e, (short)0, 2 * A.cs * es, kBufferDword3);
    const auto Rp = __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, 2 * co, kBufferDword3);
    const auto Rn = __builtin_amdgcn_make_buffer_rsrc((void*)pn, (short)0, 2 * co, kBufferDword3);
    const auto Rq = __builtin_amdgcn_make_buffer_rsrc((void*)q_, (short)0, 2 * co, kBufferDword3);
    const auto Rk = __builtin_amdgcn_make_buffer_rsrc((void*)(MODE ? beta : p), (short)0, 2 * co, kBufferDword3);

    // by colour and plane modulo 4
    E ev[2][4] = {};
    double po[2][4] = {}, be[2][4] = {}, pv[2][4] = {}, zl[2][4] = {};
    Sum2 pq;

    auto load = [&](auto ph, int q) {
        constexpr int PH = decltype(ph)::value;
        int z = min(q, zmax);
        if (perz) {
            z += z < 0 ? n2 : 0;
            z -= z >= n2 ? n2 : 0;
        }
        const int zo = z * pl + pl, ze = z * A.GH * es + A.GH * es;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const bool isA = ((c + PH) & 1) == 0;
            ev[c][PH] = Raw<E>::ld(Re, isA ? eA : eB, ze + c * A.cs * es);
            po[c][PH] = Raw<double>::ld(Rp, isA ? vA : vB, zo + c * co);
            if constexpr (MODE != 0) be[c][PH] = Raw<double>::ld(Rk, isA ? vA : vB, zo + c * co);
        }
    };
    struct Three { double x, d, u; };
    auto near = [&](int buf, bool isA) {
        const double* hp = lds + buf * NT;
        return Three{hp[isA ? sxA : sxB], hp[sdn], hp[sup]};
    };
    auto step = [&](auto ph, int q) {
        constexpr int PH = decltype(ph)::value, P1 = (PH + 3) & 3, P2 = (PH + 2) & 3;  // planes q, q-1, q-2
        constexpr int s0 = PH & 1, s1 = s0 ^ 1;
        Three np[2], nk[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {  // neighbours of plane q-1's cells, of the other colour
            const bool isA = ((c + P1) & 1) == 0;
            np[c] = near(bP + 2 * (1 - c) + s1, isA);
            if constexpr (MODE != 0) nk[c] = near(bK + 2 * (1 - c) + s1, isA);
        }
        const bool mine = q >= z0 && q < zlim;
        const int zn = mine ? q * pl + pl : 0;  // (see kOffPastBox)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const bool isA = ((c + PH) & 1) == 0;
            pv[c][PH] = (double)ev[c][PH] + bs * po[c][PH];
            lds[(bP + 2 * c + s0) * NT + tid] = pv[c][PH];
            Raw<double>::st(Rn, mine ? (isA ? wA : wB) : kOffPastBox, zn + c * co, pv[c][PH]);
            if constexpr (MODE != 0) {
                lds[(bK + 2 * c + s0) * NT + tid] = be[c][PH];
                double lo = be[1 - c][P1], hi = be[c][PH];
                lo = !perz && q == 0 ? hi : lo;
                hi = !perz && q == n2 ? lo : hi;
                zl[c][PH] = harm(lo, hi);
            }
        }
        const bool mine1 = q - 1 >= z0 && q - 1 < zlim;
        const int zq = mine1 ? q * pl : 0;
        const double kin = MODE ? harm(be[0][P1], be[1][P1]) : 1.0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const bool isA = ((c + P1) & 1) == 0, fx = isA ? fxA : fxB;
            const double v = pv[c][P1], g = -v;
            const double x = fx ? g : np[c].x, d = fyl ? g : np[c].d, u = fyr ? g : np[c].u;
            const double zm = !perz && q == 1 ? g : pv[1 - c][P2], zp = !perz && q == n2 ? g : pv[1 - c][PH];
            double su, sb;
            if constexpr (MODE == 0) {
                su = ((pv[1 - c][P1] + x) + (d + u)) + (zm + zp);
                sb = 6.0;
            } else {
                const double b = be[c][P1];
                const double ko = harm(b, fx ? b : nk[c].x), kd = harm(fyl ? b : nk[c].d, b),
                             ku = harm(b, fyr ? b : nk[c].u), kl = zl[c][P1], kh = zl[1 - c][PH];
                su = ((kin * pv[1 - c][P1] + ko * x) + (kd * d + ku * u)) + (kl * zm + kh * zp);
                sb = ((kin + ko) + (kd + ku)) + (kl + kh);
            }
            sb = sb + dg;
            const double qv = (su - sb * v) * ih2;
            Raw<double>::st(Rq, mine1 ? (isA ? wA : wB) : kOffPastBox, zq + c * co, qv);
            pq.dot(own && mine1 ? v : 0.0, own && mine1 ? qv : 0.0);
        }
    };
    load(integral_constant<int, 0>(), zs);
    load(integral_constant<int, 1>(), zs + 1);
    for (int qb = zs;; qb += 4) {
#define BXMG_STEP(PH)                                            \
    {                                                            \
        const int q = qb + PH;                                   \
        if (q >= zend) break;                                    \
        load(integral_constant<int, (PH + 2) & 3>(), q + 2);     \
        step(integral_constant<int, PH>(), q);                   \
        lds_barrier();                                           \
    }
        BXMG_STEP(0) BXMG_STEP(1) BXMG_STEP(2) BXMG_STEP(3)
#undef BXMG_STEP
    }
    block_sum2(pq, lds);
    if (tid == 0) store_sums(partials, blk, pq, Sum2{});
}

std::vector<int> piece_sizes(int cells, int unit, bool sparse) {
    const int u = cells / unit;
    std::vector<int> out;
    for (int p = 1; p <= u; p += sparse && p >= 16 ? p / 8 : 1) {
        const int size = (u + p - 1) / p * unit;
        if (out.empty() || out.back() != size) out.push_back(size);
    }
    return out;
}

// The blocks of k_kr_direction: the split with the fewest columns and planes
// read per cell that still gives every CU two rounds of two blocks.
SweepPlan plan_direction(const RBox& B, const int per[3]) {
    SweepPlan best;
    int n[3];
    for (int d = 0; d < 3; ++d) {
        n[d] = B.hi[d] - B.lo[d] + 1;
        if (n[d] % 2 || n[d] < 4 || (B.lo[d] & 1)) return best;
    }
    const int nm = n[0] / 2;
    double cost = 1e30;
    const std::vector<int> ys = piece_sizes(n[1], 1), zs = piece_sizes(n[2], 2, true);
    for (int XM : piece_sizes(nm, 1)) {
        const int hm = XM == nm ? 0 : 1, RM = XM + 2 * hm;
        if (XM < 8 && XM < nm) break;
        if (RM > kDirThreads) continue;
        for (int TY : ys) {
            const int hy = TY == n[1] ? 0 : 1, cols = RM * (TY + 2 * hy);
            if (cols > kDirThreads) continue;
            const int nbx = (nm + XM - 1) / XM, nby = (n[1] + TY - 1) / TY;
            for (int ZC : zs) {
                const int nbz = (n[2] + ZC - 1) / ZC;
                const long long blocks = (long long)nbx * nby * nbz, rounds = (blocks + 511) / 512;
                const double c = (double)rounds * (ZC + 4) * (1.0 + (cols + 63) / 64) + 1e-3 * (double)blocks;
                if (c < cost) {
                    cost = c;
                    best.nt = kDirThreads;
                    best.threads = (cols + 63) / 64 * 64;
                    best.blocks = (int)blocks;
                    SweepArgs& A = best.args;
                    A.RM = RM; A.RY = TY + 2 * hy; A.hm = hm; A.hy = hy;
                    A.XM = XM; A.TY = TY; A.ZC = ZC;
                    A.nbx = nbx; A.nby = nby; A.nbz = nbz;
                }
            }
        }
    }
    SweepArgs& A = best.args;
    for (int d = 0; d < 3; ++d) { A.n[d] = n[d]; A.per[d] = per[d]; }
    A.H = B.H;
    A.GH = B.H * B.G[1];
    A.cs = (int)B.cstride;
    A.pid = B.pid;
    A.h = B.h;
    A.a = B.a;
    return best;
}

template <class E>
hipError_t launch_kr_direction(hipStream_t s, const SweepPlan& P, const E* e, const double* p, double* pn,
                               const double* beta, double* q, const KrylovScalars* sc, double* partials,
                               const int* active) {
    const dim3 G(P.blocks), B(P.threads);
    if (beta)
        hipLaunchKernelGGL((k_kr_direction<E, 1>), G, B, 0, s, P.args, e, p, pn, beta, q, sc, partials, active);
    else
        hipLaunchKernelGGL((k_kr_direction<E, 0>), G, B, 0, s, P.args, e, p, pn, beta, q, sc, partials, active);
    return hipGetLastError();
}
template hipError_t launch_kr_direction<float>(hipStream_t, const SweepPlan&, const float*, const double*, double*,
                                               const double*, double*, const KrylovScalars*, double*, const int*);
template hipError_t launch_kr_direction<double>(hipStream_t, const SweepPlan&, const double*, const double*, double*,
                                                const double*, double*, const KrylovScalars*, double*, const int*);

// Blocks of a level: every split of its rows and planes into blocks of at
// most 1024 columns is priced as (rounds of blocks over the CUs) x (steps of a
// block) x (time of a step) and the cheapest taken.  A hierarchy is planned on
// its first solve, so each size of a piece is priced once: 0.4 ms for the levels
// of 512^3, 52 with every number of pieces (256^3: 0.2 and 11).  A step's time in
// clocks is linear in the waves on a CU (fitted to timings of every split of
// levels of 32^3 to 128^3: the plans are within 10 % of the best one there).  It
// knows neither bytes nor interpolation, so the price of large levels is too low
// (at 256^3 about 92 us a launch, for 160 and 217); their splits were not timed.
SweepPlan plan_sweep(const int n[3], const int per[3], int kind, bool zero, bool f32, int mode, int cus, int ntmax) {
    SweepPlan best;
    const bool res = kind == kSweepRestrict || kind == kSweepNorm;
    const int halo = (res ? 5 : 4) - (zero && mode != 1 ? 1 : 0);
    const int lead = ((halo + 1) & ~1) + (kind == kSweepRestrict ? 6 : res ? 5 : 4);
    const int nm = n[0] / 2;
    // (the FP64 forms and those with coefficients keep up to 168 registers a
    // thread: at most 12 waves, 8 where those would spill)
    ntmax = std::min(ntmax, f32 && mode == 0 ? 1024 : mode == 2 && kind != kSweepRestrict ? 512 : 768);
    double cost = 1e30;
    const std::vector<int> ys = piece_sizes(n[1], 2), zs = piece_sizes(n[2], 2, true);
    for (int XM : piece_sizes(nm, 1)) {
        const bool wx = XM == nm;
        if (XM < 4 && !wx) break;
        const int hm = wx ? 0 : (halo + 1) / 2, RM = XM + 2 * hm;
        if (RM > ntmax) continue;
        for (int TY : ys) {
            const bool wy = TY == n[1];
            const int hy = wy ? 0 : halo, RY = TY + 2 * hy;
            // (after the coarse levels a block also needs a thread per coarse column)
            const int cols = std::max(RM * RY, kind == kSweepRestrict ? 0 : (RM + 2) * (RY / 2 + 3));
            if (cols > ntmax) continue;
            const int nt = cols <= 256 ? 256 : cols <= 512 ? 512 : cols <= 768 ? 768 : 1024;
            const int nbx = (nm + XM - 1) / XM, nby = (n[1] + TY - 1) / TY;
            const int fit = mode ? (nt == 256 ? 3 : 1) : nt == 256 ? 5 : nt == 512 ? 2 : 1;  // blocks a CU holds (registers)
            for (int ZC : zs) {
                const int nbz = (n[2] + ZC - 1) / ZC;
                const long long blocks = (long long)nbx * nby * nbz;
                const long long per_cu = (blocks + cus - 1) / cus;
                const long long rounds = (per_cu + fit - 1) / fit;
                const int waves = (int)std::min<long long>(per_cu, fit) * ((cols + 63) / 64);
                const double step = mode ? 700.0 + 280.0 * waves : f32 ? 600.0 + 80.0 * waves : 550.0 + 115.0 * waves;
                const double c = rounds * (ZC + lead) * step + 1e-3 * blocks;
                if (c < cost) {
                    cost = c;
                    best.nt = nt;
                    best.threads = (cols + 63) / 64 * 64;
                    best.blocks = (int)blocks;
                    SweepArgs& A = best.args;
                    A.RM = RM; A.RY = RY; A.hm = hm; A.hy = hy;
                    A.XM = XM; A.TY = TY; A.ZC = ZC;
                    A.nbx = nbx; A.nby = nby; A.nbz = nbz;
                }
            }
        }
    }
    for (int d = 0; d < 3; ++d) { best.args.n[d] = n[d]; best.args.per[d] = per[d]; }
    return best;
}

SweepPlan plan_sweep_level(const RBox& B, const RBox& Q, const int per[3], int kind, bool zero, bool f32, int mode,
                           int cus, int ntmax) {
    int n[3];
    for (int d = 0; d < 3; ++d) {
        n[d] = B.hi[d] - B.lo[d] + 1;
        if (n[d] % 2 || n[d] < 4 || (B.lo[d] & 1)) return SweepPlan{};
    }
    SweepPlan P = plan_sweep(n, per, kind, zero, f32, mode, cus, ntmax);
    SweepArgs& A = P.args;
    A.H = B.H;
    A.GH = B.H * B.G[1];
    A.cs = (int)B.cstride;
    A.cH = Q.H;
    A.cGH = Q.H * Q.G[1];
    A.ccs = (int)Q.cstride;
    A.cpar = (Q.lo[0] + Q.lo[1] + Q.lo[2]) & 1;
    A.pid = B.pid;
    A.h = B.h;
    A.a = B.a;
    return P;
}

template <class T>
hipError_t launch_sweep(hipStream_t s, const SweepPlan& P, bool zero, bool post, int kind, const T* uin, T* uout,
                        const T* f, T* cf, double* acc, double* partials, const int* active, int mode, const T* beta,
                        const FaceArrays<T>* fat, const T* ec, int order) {
    const dim3 G((unsigned)P.blocks);
    SweepArgs args = P.args;
    args.order = order;
    constexpr bool F64 = std::is_same<T, double>::value;
#define BXMG_SW(NT, ZERO, KIND, POST, MODE)                                                                       \
    hipLaunchKernelGGL((k_sweep<T, NT, ZERO, KIND, POST, false, MODE>), G, dim3(P.threads), 0, s, args,           \
                       (const SweepArgs*)nullptr, (const int2*)nullptr, uin, uout, f, cf, acc, partials, active, \
                       beta, fat, ec)
#define BXMG_SWN(ZERO, KIND, POST, MODE)                   \
    if (P.nt == 256) BXMG_SW(256, ZERO, KIND, POST, MODE); \
    else if (P.nt == 512) BXMG_SW(512, ZERO, KIND, POST, MODE); \
    else if (MODE == 2 && POST) return hipErrorInvalidValue; \
    else if (P.nt == 768) BXMG_SW((MODE == 2 && POST ? 512 : 768), ZERO, KIND, POST, MODE); \
    else if constexpr (!F64 && MODE == 0) BXMG_SW(1024, ZERO, KIND, POST, MODE); \
    else return hipErrorInvalidValue
#define BXMG_SWM(ZERO, KIND, POST)                                \
    if (mode == 0) { BXMG_SWN(ZERO, KIND, POST, 0); }             \
    else if constexpr (!F64) {                                    \
        if (mode == 1) { BXMG_SWN(ZERO, KIND, POST, 1); }         \
        else { BXMG_SWN(ZERO, KIND, POST, 2); }                   \
    } else return hipErrorInvalidValue
    if (kind == kSweepRestrict && !post && zero) {
        BXMG_SWM(true, kSweepRestrict, false);
    } else if (kind == kSweepRestrict && !post && F64) {  // (FP32 levels start from zero)
        if constexpr (F64) { BXMG_SWM(false, kSweepRestrict, false); }
    } else if (kind == kSweepNorm && post && F64) {
        if constexpr (F64) { BXMG_SWM(false, kSweepNorm, true); }
    } else if (kind == kSweepAdd && post && !F64 && mode < 2) {  // (a level 0)
        if constexpr (!F64) {
            if (mode == 0) { BXMG_SWN(false, kSweepAdd, true, 0); }
            else { BXMG_SWN(false, kSweepAdd, true, 1); }
        }
    } else if (kind == kSweepPlain && post) {
        BXMG_SWM(false, kSweepPlain, true);
    } else {
        return hipErrorInvalidValue;
    }
#undef BXMG_SWM
#undef BXMG_SWN
#undef BXMG_SW
    return hipGetLastError();
}
template hipError_t launch_sweep<double>(hipStream_t, const SweepPlan&, bool, bool, int, const double*, double*,
                                         const double*, double*, double*, double*, const int*, int, const double*,
                                         const FaceArrays<double>*, const double*, int);
template hipError_t launch_sweep<float>(hipStream_t, const SweepPlan&, bool, bool, int, const float*, float*,
                                        const float*, float*, double*, double*, const int*, int, const float*,
                                        const FaceArrays<float>*, const float*, int);

hipError_t launch_sweep_jobs(hipStream_t s, const SweepArgs* jobs, const int2* where, int blocks, int threads,
                             int kind, const float* uin, float* uout, const float* f, float* cf, double* acc,
                             const int* active, const float* ec) {
    if (blocks <= 0) return hipSuccess;
    if (threads > kSweepJobThreads) return hipErrorInvalidValue;
#define BXMG_SWJ(ZERO, KIND, POST)                                                                               \
    hipLaunchKernelGGL((k_sweep<float, kSweepJobThreads, ZERO, KIND, POST, true, 0>), dim3(blocks), dim3(threads), 0, s, \
                       SweepArgs{}, jobs, where, uin, uout, f, cf, acc, (double*)nullptr, active, (const float*)nullptr, \
                       (const FaceArrays<float>*)nullptr, ec)
    if (kind == kSweepRestrict) BXMG_SWJ(true, kSweepRestrict, false);
    else if (kind == kSweepPlain) BXMG_SWJ(false, kSweepPlain, true);
    else if (kind == kSweepAdd) BXMG_SWJ(false, kSweepAdd, true);
    else return hipErrorInvalidValue;
#undef BXMG_SWJ
    return hipGetLastError();
}

}  // namespace bxmg
