// Nodal-centred Poisson solver (the framework's other linear-solver family,
// paper Section 2): V-cycles over node-centred data of the whole domain.
//
// On a domain of n_d cells of width h per direction the nodes sit at
// x = i h, i = 0 .. n_d.  The caller's arrays are F-order over the
// (n_0+1)(n_1+1)(n_2+1) nodes; every level is held colour-split inside the
// solver: node (i, j, k) of colour c = (i + j + k) & 1 in colour block c,
// row k (n_1+1) + j, slot i >> 1 (rows of (n_0+2)/2 slots), so a colour
// sweep streams the other colour, its own right-hand side and its own
// writes.  A homogeneous-Dirichlet
// direction keeps its boundary nodes at 0 (they are not unknowns); in a
// periodic direction node n_d is node 0: the kernels read neighbours
// through the wrapped index, and the copies n_d are refreshed only in the
// solution handed back.  Operator (L u)_i = (sum of the 6 neighbours - 6 u_i)
// / h^2; red-black Gauss-Seidel on node parity; full-weighting restriction
// (weights 1/2 at the node, 1/4 at +-1 per direction); trilinear
// prolongation; FP64 CG bottom in one workgroup.  Coarse node I is fine node
// 2I; levels halve while every n_d is even and > 2.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cmath>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "bxmg_device.h"
#include "bxmg_host.h"

namespace bxmg {
namespace nodal {

struct NLev {
    int n[3];    // cells per direction (nodes 0..n)
    int per[3];
    double h;
    long long size;   // nodes, (n0+1)(n1+1)(n2+1)
    int H;            // slots per colour row, (n0+2)/2
    long long cs;     // colour block stride (elements)
    long long alloc;  // elements of a level array, 2 cs
};

// offset of node (i, j, k) in the colour-split level array
__host__ __device__ inline long long nidx(const NLev& L, int i, int j, int k) {
    return ((i + j + k) & 1) * L.cs + (long long)((k * (L.n[1] + 1) + j) * L.H + (i >> 1));
}

// node (i, j, k) of the g-th node in F order (x fastest)
__device__ __forceinline__ void coords(const NLev& L, long long g, int& i, int& j, int& k) {
    const int nx = L.n[0] + 1, ny = L.n[1] + 1;
    const long long r = g / nx;
    i = (int)(g - r * nx);
    j = (int)(r % ny);
    k = (int)(r / ny);
}

__device__ __forceinline__ bool unknown(const NLev& L, int i, int j, int k) {
    const int c[3] = {i, j, k};
#pragma unroll
    for (int d = 0; d < 3; ++d)
        if (L.per[d] ? c[d] == L.n[d] : (c[d] == 0 || c[d] == L.n[d])) return false;
    return true;
}

__device__ __forceinline__ int wrap(const NLev& L, int d, int c) {
    if (!L.per[d]) return c;
    return c < 0 ? c + L.n[d] : (c >= L.n[d] ? c - L.n[d] : c);
}

// sum of the 6 neighbours, ((x- + x+) + (y- + y+)) + (z- + z+)
__device__ __forceinline__ double nsum(const NLev& L, const double* __restrict__ u, int i, int j, int k) {
    const double xm = u[nidx(L, wrap(L, 0, i - 1), j, k)], xp = u[nidx(L, wrap(L, 0, i + 1), j, k)];
    const double ym = u[nidx(L, i, wrap(L, 1, j - 1), k)], yp = u[nidx(L, i, wrap(L, 1, j + 1), k)];
    const double zm = u[nidx(L, i, j, wrap(L, 2, k - 1))], zp = u[nidx(L, i, j, wrap(L, 2, k + 1))];
    return ((xm + xp) + (ym + yp)) + (zm + zp);
}

__device__ __forceinline__ void block_sum2(double& a, double& b, double* sh) {
    for (int o = 32; o > 0; o >>= 1) {
        a = a + __shfl_xor(a, o);
        b = b + __shfl_xor(b, o);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) { sh[2 * wid] = a; sh[2 * wid + 1] = b; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        a = sh[0];
        b = sh[1];
        for (int w = 1; w < nw; ++w) { a = a + sh[2 * w]; b = b + sh[2 * w + 1]; }
    }
}

constexpr int kNB = 256;

// Level kernels walk planes: grid (plane blocks, plane groups), a thread
// takes one (x, y) position of its planes.  Interior nodes read their six
// neighbours directly (x from the other colour's slots (i -+ 1) >> 1, y and z
// from the other colour's rows at slot i >> 1); the others go through the
// wrapped index.
constexpr int kKZ = 8;

// the six neighbours of interior node (i, j, k), ((x- + x+) + (y- + y+)) + (z- + z+)
__device__ __forceinline__ double nsum_in(const NLev& L, const double* __restrict__ u, int i, int j, int k) {
    const int c = (i + j + k) & 1;
    const long long o = (1 - c) * L.cs + (long long)((k * (L.n[1] + 1) + j) * L.H);
    const long long m = o + (i >> 1), sy = L.H, sz = (long long)L.H * (L.n[1] + 1);
    return ((u[o + ((i - 1) >> 1)] + u[o + ((i + 1) >> 1)]) + (u[m - sy] + u[m + sy])) + (u[m - sz] + u[m + sz]);
}

// no neighbour through a wrap: in a periodic direction node n_d - 1 reads
// node 0 through the wrapped index (the copy n_d is refreshed only at the
// end), so it is not interior
__device__ __forceinline__ bool interior(const NLev& L, int i, int j, int k) {
    return i > 0 && i < L.n[0] - L.per[0] && j > 0 && j < L.n[1] - L.per[1] && k > 0 && k < L.n[2] - L.per[2];
}

// one colour: a thread per colour node of a row position (i = 2t + parity)
__global__ void __launch_bounds__(kNB) k_nd_gs(NLev L, double* __restrict__ u, const double* __restrict__ f,
                                              int colour, int kz) {
    const uint3 bk = xcd_block();
    const int hx = (L.n[0] + 2) / 2, ny = L.n[1] + 1;
    const int t = bk.x * kNB + threadIdx.x;
    if (t >= hx * ny) return;
    const int tx = t % hx, j = t / hx;
    const int k0 = bk.y * kz, k1 = min(k0 + kz - 1, L.n[2]);
    const double h2 = L.h * L.h;
    for (int k = k0; k <= k1; ++k) {
        const int i = 2 * tx + ((colour - j - k) & 1);
        if (i > L.n[0] || !unknown(L, i, j, k)) continue;
        const long long q = nidx(L, i, j, k);
        const double su = interior(L, i, j, k) ? nsum_in(L, u, i, j, k) : nsum(L, u, i, j, k);
        u[q] = (su - h2 * f[q]) / 6.0;
    }
}

// r = f - L u at the unknowns, 0 at the other nodes; partial (max, sum r^2,
// non-finite count) per block
__global__ void __launch_bounds__(kNB) k_nd_resid(NLev L, const double* __restrict__ u,
                                                 const double* __restrict__ f, double* __restrict__ r,
                                                 double* __restrict__ partials, int kz) {
    __shared__ double sh[3 * (kNB / 64)];
    const uint3 bk = xcd_block();
    const int hx = (L.n[0] + 2) / 2, ny = L.n[1] + 1;
    const int t = bk.x * kNB + threadIdx.x;
    const double ih2 = 1.0 / (L.h * L.h);
    double mx = 0.0, s2 = 0.0, bad = 0.0;
    if (t < hx * ny) {
        // a thread per row slot, the node of each colour in it
        const int tx = t % hx, j = t / hx;
        const int k0 = bk.y * kz, k1 = min(k0 + kz - 1, L.n[2]);
        for (int k = k0; k <= k1; ++k)
          for (int c = 0; c < 2; ++c) {
            const int i = 2 * tx + ((c - j - k) & 1);
            if (i > L.n[0]) continue;
            const long long q = nidx(L, i, j, k);
            double rv = 0.0;
            if (unknown(L, i, j, k)) {
                const double su = interior(L, i, j, k) ? nsum_in(L, u, i, j, k) : nsum(L, u, i, j, k);
                rv = f[q] - (su - 6.0 * u[q]) * ih2;
                const double a = fabs(rv);
                if (!(a <= 1.7976931348623157e308)) bad += 1.0;
                else mx = fmax(mx, a);
                s2 = s2 + rv * rv;
            }
            r[q] = rv;
          }
    }
    for (int o = 32; o > 0; o >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, o));
        s2 = s2 + __shfl_xor(s2, o);
        bad = bad + __shfl_xor(bad, o);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) { sh[3 * wid] = mx; sh[3 * wid + 1] = s2; sh[3 * wid + 2] = bad; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kNB / 64; ++w) { mx = fmax(mx, sh[3 * w]); s2 = s2 + sh[3 * w + 1]; bad = bad + sh[3 * w + 2]; }
        const int blk = bk.y * gridDim.x + bk.x;
        partials[3 * blk] = mx;
        partials[3 * blk + 1] = s2;
        partials[3 * blk + 2] = bad;
    }
}

// Streaming smoother: two red-black sweeps of a level and the residual after
// them in one pass (the cell-centred one, bxmg_sweep.hip, describes the
// scheme: a block walks a column of the level in z, the four half-sweeps and
// the residual one plane behind each other, values in registers and the last
// planes' in LDS).  A thread holds the pair of nodes (2m, 2m + 1) of a row; a
// boundary node keeps its value through all stages, so no neighbour needs a
// special case, and node n_d is written by the block that owns node n_d - 1.
// ZERO: the sweeps start from u = 0, which is not read; otherwise colour 0 is
// read at boundary nodes only.  KIND: 0 no residual, 1 the residual of the
// unknowns into r, 2 its norms (3 partials per block).  uin and uout differ.
// POST: the sweeps after the coarse levels; the correction e of colour 1 is
// interpolated as it enters, from the coarse planes of the block's columns in
// LDS (two at a time, a thread carrying one value of the next).
// 256^3, FP64: sweeps and residual 165 us, sweeps with the interpolation and the
// norms 195, against 4 x 56 + 122 and 159 + 4 x 56 + 122 in launches of their
// own; 128^3 27 and 28 us, against 4 x 9.0 + 17 and 12 + 4 x 9.0.  The arrays
// alone (u, f in, u, r out) take about 100 us at the copy rate.
struct NSweep {
    int nt = 0, threads = 0, blocks = 0;
    int RM, RY;          // columns of a block with its halo: pairs, rows
    int hm, hy;          // the halo below: pairs, rows (0: the block spans the level there)
    int XM, TY, ZC;      // what a block owns
    int nbx, nby, nbz;
    int cH, cpl, ccs;    // the coarse level: row, plane and colour block (elements)
};
template <int NT, bool ZERO, int KIND, bool POST>
__global__ void __launch_bounds__(NT) k_nd_sweep(NLev L, NSweep A, const double* __restrict__ uin,
                                                double* __restrict__ uout, const double* __restrict__ f,
                                                double* __restrict__ r, double* __restrict__ partials,
                                                const double* __restrict__ e) {
    using std::integral_constant;
    constexpr bool RES = KIND != 0;
    constexpr int bB0 = 0, bR1 = 2, bB2 = 4, bR3 = 6, bB4 = 10, bC = RES ? 12 : 10;
    __shared__ double lds[(bC + (POST ? 2 : 0)) * NT];
    const int tid = threadIdx.x;
    int blk = blockIdx.x;
    {
        const int nb = gridDim.x;
        if ((nb & 7) == 0) blk = (blk & 7) * (nb >> 3) + (blk >> 3);
    }
    const int bx = blk % A.nbx, byz = blk / A.nbx;
    const int by = byz % A.nby, bz = byz / A.nby;
    const int nm = L.n[0] >> 1, n1 = L.n[1], n2 = L.n[2];
    const bool perx = L.per[0] != 0, pery = L.per[1] != 0, perz = L.per[2] != 0;
    const int ty = tid / A.RM, tm = tid - ty * A.RM;
    const int mr = bx * A.XM - A.hm + tm, yr = by * A.TY - A.hy + ty;
    int m = mr, y = yr;
    bool in = ty < A.RY;
    if (perx) { m %= nm; m += m < 0 ? nm : 0; } else in = in && m >= 0 && m <= nm;
    if (pery) { y %= n1; y += y < 0 ? n1 : 0; } else in = in && y >= 0 && y <= n1;
    const int x1 = min((bx + 1) * A.XM, nm), y1 = min((by + 1) * A.TY, n1);
    const bool own = in && mr >= bx * A.XM && (mr < x1 || (!perx && mr == nm && x1 == nm)) && yr >= by * A.TY &&
                     (yr < y1 || (!pery && yr == n1 && y1 == n1));
    const int z0 = bz * A.ZC, zlim = min(z0 + A.ZC, n2);
    constexpr int kHalo = (RES ? 5 : 4) - (ZERO ? 1 : 0), kFirst = (kHalo + 1) & ~1;
    const int zs = perz ? z0 - kFirst : max(0, z0 - kFirst);
    const int zend = zlim + 5;
    const int zmax = perz ? zlim + 4 : min(zlim + 4, n2);
    const bool top = !perz && zlim == n2;  // also writes plane n2
    // in a plane of parity p the colour-c node of the pair is 2m + o, o = (c + y
    // + p) & 1; "A" is the node with o = yo
    const int yo = y & 1;
    const bool wx = perx && A.hm == 0, wy = pery && A.hy == 0;
    const int sl = tm > 0 ? tid - 1 : wx ? tid + A.RM - 1 : tid;
    const int sr = tm < A.RM - 1 ? tid + 1 : wx ? tid - (A.RM - 1) : tid;
    const int sdn = !in ? tid : ty > 0 ? tid - A.RM : wy ? tid + (A.RY - 1) * A.RM : tid;
    const int sup = !in ? tid : ty < A.RY - 1 ? tid + A.RM : wy ? tid - (A.RY - 1) * A.RM : tid;
    const int sxA = !in ? tid : yo ? sr : sl;
    const int sxB = !in ? tid : yo ? sl : sr;
    // boundary nodes (the slot beyond node n_0 counts as one)
    const bool fy = in && !pery && (y == 0 || y == n1);
    const bool fl = in && !perx && m == 0, fr_ = in && !perx && m == nm;
    const bool fixA = fy || fr_ || (fl && yo == 0), fixB = fy || fr_ || (fl && yo == 1);
    const bool edge_xy = __ballot(fixA || fixB) != 0;
    const int v = in ? (y * L.H + m) * 8 : kOffPastBox;
    const int co = (int)L.cs * 8, pl = L.H * (n1 + 1) * 8;
    const int w = own ? v : kOffPastBox;
    const double h2 = uniform(L.h * L.h), ih2 = uniform(1.0 / (L.h * L.h));
    const Recip<double> r6(6.0);
    const int bytes = 2 * co;
    // POST: the block's coarse columns, one per thread (offset in a plane, parity
    // of I + J), and the pair's place among them
    const int y0 = by * A.TY - A.hy, CW = A.RM + 1;
    int ci = kOffPastBox, cp = 0, ic = 0;
    if constexpr (POST) {
        const int cy = tid / CW, nr = ((y0 + A.RY - 1) >> 1) + 2 - (y0 >> 1);
        auto node = [](int c, int n, bool per) {
            if (!per) return min(max(c, 0), n);
            c %= n;
            return c < 0 ? c + n : c;
        };
        const int I = node(bx * A.XM - A.hm + tid - cy * CW, nm, perx), J = node((y0 >> 1) + cy, n1 >> 1, pery);
        if (cy < nr) ci = (J * A.cH + (I >> 1)) * 8;
        cp = (I + J) & 1;
        ic = in ? ((yr >> 1) - (y0 >> 1)) * CW + tm : 0;
    }
    const auto Rc = __builtin_amdgcn_make_buffer_rsrc((void*)(POST ? e : f), (short)0, POST ? 2 * A.ccs * 8 : bytes,
                                                      kBufferDword3);
    auto load_coarse = [&](int K) {  // of plane K (wrapped; past the last one of a Dirichlet level: any)
        const int nk = n2 >> 1;
        if (perz) {
            K = K < 0 ? K + nk : K >= nk ? K - nk : K;
            K = K < 0 ? K + nk : K >= nk ? K - nk : K;
        }
        K = min(max(K, 0), nk);
        return Raw<double>::ld(Rc, ci + ((cp + K) & 1) * (A.ccs * 8), K * A.cpl * 8);
    };
    double cr = 0.0;
    const auto Ru = __builtin_amdgcn_make_buffer_rsrc((void*)(ZERO ? f : uin), (short)0, bytes, kBufferDword3);
    const auto Rf = __builtin_amdgcn_make_buffer_rsrc((void*)f, (short)0, bytes, kBufferDword3);
    const auto Ro = __builtin_amdgcn_make_buffer_rsrc((void*)uout, (short)0, bytes, kBufferDword3);
    const auto Rr = __builtin_amdgcn_make_buffer_rsrc((void*)(KIND == 1 ? r : uout), (short)0, bytes, kBufferDword3);

    double r0[8], b0[8], r1[8], b2[8], r3[8], b4[8], f0[8], f1[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        r0[k] = 0.0; b0[k] = 0.0; r1[k] = 0.0; b2[k] = 0.0;
        r3[k] = 0.0; b4[k] = 0.0; f0[k] = 0.0; f1[k] = 0.0;
    }
    double mx = 0.0, s2 = 0.0;
    int nbad = 0;

    auto load = [&](auto ph, int q) {
        constexpr int PH = decltype(ph)::value;
        int z = min(q, zmax);
        if (perz) {
            z += z < 0 ? n2 : 0;
            z += z < 0 ? n2 : 0;
            z -= z >= n2 ? n2 : 0;
            z -= z >= n2 ? n2 : 0;
        }
        const int zo = z * pl;
        f0[PH] = Raw<double>::ld(Rf, v, zo);
        f1[PH] = Raw<double>::ld(Rf, v, zo + co);
        if constexpr (!ZERO) {
            b0[PH] = Raw<double>::ld(Ru, v, zo + co);
            const bool fz = !perz && (z == 0 || z == n2);
            r0[PH] = 0.0;  // (or each slot's last value would stay live)
            if (edge_xy || fz) {
                const bool fix = fz || ((PH & 1) ? fixB : fixA);
                r0[PH] = Raw<double>::ld(Ru, fix ? v : kOffPastBox, zo);
            }
        }
    };

    auto step = [&](auto ph, auto edge, int q) {
        constexpr int PH = decltype(ph)::value;
        constexpr bool EDGE = decltype(edge)::value != 0;
#define RS(d) ((PH - (d) + 16) & 7)              /* ring slot of plane q - d */
#define ISA(d, c) ((((c) + PH - (d)) & 1) == 0)  /* its colour-c node is at o = yo */
        struct Three { double x, d, u; };
        auto near = [&](int buf, bool isA) {
            const double* hp = lds + buf * NT;
            return Three{hp[isA ? sxA : sxB], hp[sdn], hp[sup]};
        };
        auto fixed = [&](int d, bool isA) {  // in plane q - d
            return (isA ? fixA : fixB) || (!perz && (q == d || q == d + n2));
        };
        auto relax = [&](int d, bool isA, double own_o, Three n, double zm, double zp, double fv, double old) {
            const double x = r6.div(((own_o + n.x) + (n.d + n.u)) + (zm + zp) - h2 * fv);
            if constexpr (EDGE) return fixed(d, isA) ? old : x;
            else return x;
        };
        if constexpr (POST) {
            // colour 1 of plane q: its row's parity decides between 2 coarse nodes
            // along x or y (even planes), 2 along z or all 8 (odd ones)
            const double* a = lds + (bC + ((PH >> 1) & 1)) * NT + ic;
            double v;
            if constexpr ((PH & 1) == 0) {
                v = (a[0] + a[yo ? CW : 1]) * 0.5;
            } else {
                const double* b = lds + (bC + (((PH >> 1) + 1) & 1)) * NT + ic;
                const double two = (a[0] + b[0]) * 0.5;
                const double all =
                    (((((((a[0] + a[1]) + a[CW]) + a[CW + 1]) + b[0]) + b[1]) + b[CW]) + b[CW + 1]) * 0.125;
                v = yo ? all : two;
            }
            const double x = b0[RS(0)] + v;
            if constexpr (EDGE) b0[RS(0)] = fixed(0, ISA(0, 1)) ? b0[RS(0)] : x;
            else b0[RS(0)] = x;
            if constexpr ((PH & 1) == 0) {
                if (ci != kOffPastBox) lds[(bC + (((PH >> 1) + 1) & 1)) * NT + tid] = cr;
                cr = load_coarse((q >> 1) + 2);
            }
        }
        Three t1{}, t2, t3, t4, t5r{}, t5b{};
        if constexpr (!ZERO) t1 = near(bB0 + ((PH - 1) & 1), ISA(1, 0));
        t2 = near(bR1 + ((PH - 1) & 1), ISA(2, 1));
        t3 = near(bB2 + ((PH - 1) & 1), ISA(3, 0));
        t4 = near(bR3 + ((PH - 1) & 3), ISA(4, 1));
        if constexpr (RES) {
            t5r = near(bB4 + ((PH - 1) & 1), ISA(5, 0));
            t5b = near(bR3 + ((PH - 2) & 3), ISA(5, 1));
        }
        if constexpr (!ZERO) lds[(bB0 + (PH & 1)) * NT + tid] = b0[RS(0)];
        // the four half-sweeps
        if constexpr (ZERO) r1[RS(1)] = relax(1, ISA(1, 0), 0.0, Three{0.0, 0.0, 0.0}, 0.0, 0.0, f0[RS(1)], 0.0);
        else r1[RS(1)] = relax(1, ISA(1, 0), b0[RS(1)], t1, b0[RS(2)], b0[RS(0)], f0[RS(1)], r0[RS(1)]);
        lds[(bR1 + (PH & 1)) * NT + tid] = r1[RS(1)];
        b2[RS(2)] = relax(2, ISA(2, 1), r1[RS(2)], t2, r1[RS(3)], r1[RS(1)], f1[RS(2)], ZERO ? 0.0 : b0[RS(2)]);
        lds[(bB2 + (PH & 1)) * NT + tid] = b2[RS(2)];
        r3[RS(3)] = relax(3, ISA(3, 0), b2[RS(3)], t3, b2[RS(4)], b2[RS(2)], f0[RS(3)], r1[RS(3)]);
        lds[(bR3 + (PH & 3)) * NT + tid] = r3[RS(3)];
        b4[RS(4)] = relax(4, ISA(4, 1), r3[RS(4)], t4, r3[RS(5)], r3[RS(3)], f1[RS(4)], b2[RS(4)]);
        if constexpr (RES) lds[(bB4 + (PH & 1)) * NT + tid] = b4[RS(4)];
        {  // plane q-4 is final
            const int pz = q - 4;
            const bool mine = pz >= z0 && (pz < zlim || (top && pz == n2));
            const int zo = mine ? pz * pl : 0;  // (see kOffPastBox)
            Raw<double>::st(Ro, mine ? w : kOffPastBox, zo, r3[RS(4)]);
            Raw<double>::st(Ro, mine ? w : kOffPastBox, zo + co, b4[RS(4)]);
        }
        if constexpr (RES) {  // the residual of plane q-5
            const int pz = q - 5;
            const bool here = pz >= z0 && pz < zlim && (perz || pz > 0), mine = own && here;
            const int zo = here ? pz * pl : 0;
            const bool m0 = mine && !(ISA(5, 0) ? fixA : fixB), m1 = mine && !(ISA(5, 1) ? fixA : fixB);
            const double s0 = ((b4[RS(5)] + t5r.x) + (t5r.d + t5r.u)) + (b4[RS(6)] + b4[RS(4)]);
            const double s1 = ((r3[RS(5)] + t5b.x) + (t5b.d + t5b.u)) + (r3[RS(6)] + r3[RS(4)]);
            const double v0 = f0[RS(5)] - (s0 - 6.0 * r3[RS(5)]) * ih2;
            const double v1 = f1[RS(5)] - (s1 - 6.0 * b4[RS(5)]) * ih2;
            if constexpr (KIND == 1) {
                Raw<double>::st(Rr, m0 ? v : kOffPastBox, zo, v0);
                Raw<double>::st(Rr, m1 ? v : kOffPastBox, zo + co, v1);
            } else {
#pragma unroll
                for (int c = 0; c < 2; ++c) {  // (without branches: 0 adds nothing)
                    const double x = (c ? m1 : m0) ? (c ? v1 : v0) : 0.0, a = fabs(x);
                    const bool fine = a <= 1.7976931348623157e308;
                    mx = fmax(mx, fine ? a : 0.0);
                    nbad += fine ? 0 : 1;
                    s2 = s2 + x * x;
                }
            }
        }
#undef RS
#undef ISA
    };

    if constexpr (POST) {
        const double v = load_coarse(zs >> 1);
        cr = load_coarse((zs >> 1) + 1);
        if (ci != kOffPastBox) lds[bC * NT + tid] = v;
        lds_barrier();
    }
    load(integral_constant<int, 0>(), zs);
    load(integral_constant<int, 1>(), zs + 1);
    for (int qb = zs;; qb += 8) {
#define BXMG_STEP(PH)                                                           \
    {                                                                           \
        const int q = qb + PH;                                                  \
        if (q >= zend) break;                                                   \
        load(integral_constant<int, (PH + 2) & 7>(), q + 2);                    \
        if (edge_xy || (!perz && (q <= 4 || q >= n2)))                          \
            step(integral_constant<int, PH>(), integral_constant<int, 1>(), q); \
        else step(integral_constant<int, PH>(), integral_constant<int, 0>(), q); \
        lds_barrier();                                                          \
    }
        BXMG_STEP(0) BXMG_STEP(1) BXMG_STEP(2) BXMG_STEP(3)
        BXMG_STEP(4) BXMG_STEP(5) BXMG_STEP(6) BXMG_STEP(7)
#undef BXMG_STEP
    }
    if constexpr (KIND == 2) {
        double bad = (double)nbad;
        block_reduce3(mx, s2, bad, lds);  // (every read of lds ended with the last barrier)
        if (tid == 0) {
            partials[3 * (size_t)blk] = mx;
            partials[3 * (size_t)blk + 1] = s2;
            partials[3 * (size_t)blk + 2] = bad;
        }
    }
}

// The blocks of a level (as plan_sweep); nt = 0: beyond 32-bit offsets.
static NSweep plan_nd_sweep(const NLev& L, const NLev& C, bool zero, int kind, bool post) {
    NSweep best;
    if (L.alloc * 8 > 0x7fffffffLL) return best;
    const int halo = (kind ? 5 : 4) - (zero ? 1 : 0), lead = ((halo + 1) & ~1) + 5, nm = L.n[0] / 2;
    double cost = 1e30;
    const std::vector<int> ys = piece_sizes(L.n[1], 2), zs = piece_sizes(L.n[2], 2, true);
    for (int XM : piece_sizes(nm, 1)) {
        if (XM < 4 && XM < nm) break;
        const int hm = XM == nm ? 0 : (halo + 1) / 2, RM = XM == nm ? nm + (L.per[0] ? 0 : 1) : XM + 2 * hm;
        if (RM > 768) continue;
        for (int TY : ys) {
            const bool span = TY == L.n[1];
            const int hy = span ? 0 : halo, RY = span ? TY + (L.per[1] ? 0 : 1) : TY + 2 * hy;
            const int cols = std::max(RM * RY, post ? (RM + 1) * (RY / 2 + 3) : 0);
            if (cols > 768) continue;
            const int nt = cols <= 256 ? 256 : cols <= 512 ? 512 : 768;
            const int nbx = (nm + XM - 1) / XM, nby = (L.n[1] + TY - 1) / TY;
            const int fit = nt == 256 ? 3 : 1;
            for (int ZC : zs) {
                const int nbz = (L.n[2] + ZC - 1) / ZC;
                const long long blocks = (long long)nbx * nby * nbz, per_cu = (blocks + 255) / 256;
                const int waves = (int)std::min<long long>(per_cu, fit) * ((cols + 63) / 64);
                const double c = (double)((per_cu + fit - 1) / fit) * (ZC + lead) * (550.0 + 115.0 * waves) +
                                 1e-3 * (double)blocks;
                if (c < cost) {
                    cost = c;
                    best.nt = nt;
                    best.threads = (cols + 63) / 64 * 64;
                    best.blocks = (int)blocks;
                    best.RM = RM; best.RY = RY; best.hm = hm; best.hy = hy;
                    best.XM = XM; best.TY = TY; best.ZC = ZC;
                    best.nbx = nbx; best.nby = nby; best.nbz = nbz;
                }
            }
        }
    }
    best.cH = C.H;
    best.cpl = C.H * (C.n[1] + 1);
    best.ccs = (int)C.cs;
    return best;
}

template <bool ZERO, int KIND, bool POST>
static hipError_t launch_nd_sweep(hipStream_t s, const NLev& L, const NSweep& P, const double* uin, double* uout,
                                  const double* f, double* r, double* partials, const double* e) {
#define BXMG_NSW(NT)                                                                                             \
    hipLaunchKernelGGL((k_nd_sweep<NT, ZERO, KIND, POST>), dim3(P.blocks), dim3(P.threads), 0, s, L, P, uin, uout, f, \
                       r, partials, e)
    if (P.nt == 256) BXMG_NSW(256);
    else if (P.nt == 512) BXMG_NSW(512);
    else BXMG_NSW(768);
#undef BXMG_NSW
    return hipGetLastError();
}

// norms of f over the unknowns (max, sum of squares, non-finite count)
__global__ void __launch_bounds__(kNB) k_nd_fnorm(NLev L, const double* __restrict__ f,
                                                 double* __restrict__ partials) {
    __shared__ double sh[3 * (kNB / 64)];
    double mx = 0.0, s2 = 0.0, bad = 0.0;
    for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < L.size;
         g += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(L, g, i, j, k);
        if (!unknown(L, i, j, k)) continue;
        const long long q = nidx(L, i, j, k);
        const double a = fabs(f[q]);
        if (!(a <= 1.7976931348623157e308)) bad += 1.0;
        else mx = fmax(mx, a);
        s2 = s2 + f[q] * f[q];
    }
    for (int o = 32; o > 0; o >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, o));
        s2 = s2 + __shfl_xor(s2, o);
        bad = bad + __shfl_xor(bad, o);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) { sh[3 * wid] = mx; sh[3 * wid + 1] = s2; sh[3 * wid + 2] = bad; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kNB / 64; ++w) { mx = fmax(mx, sh[3 * w]); s2 = s2 + sh[3 * w + 1]; bad = bad + sh[3 * w + 2]; }
        partials[3 * blockIdx.x] = mx;
        partials[3 * blockIdx.x + 1] = s2;
        partials[3 * blockIdx.x + 2] = bad;
    }
}

// the full weighting of r at coarse unknown (I, J, K), in the order z, then y,
// then x offsets
__device__ __forceinline__ double weighted(const NLev& F, const double* r, int I, int J, int K) {
    const double w[3] = {0.25, 0.5, 0.25};
    double s = 0.0;
    for (int c = -1; c <= 1; ++c)
        for (int b = -1; b <= 1; ++b)
            for (int a = -1; a <= 1; ++a) {
                const int i = wrap(F, 0, 2 * I + a), j = wrap(F, 1, 2 * J + b), k = wrap(F, 2, 2 * K + c);
                s = s + ((w[a + 1] * w[b + 1]) * w[c + 1]) * r[nidx(F, i, j, k)];
            }
    return s;
}

// full weighting onto the coarse unknowns (0 at the other coarse nodes); the
// coarse u is zeroed on the way
__global__ void __launch_bounds__(kNB) k_nd_restrict(NLev F, const double* __restrict__ r, NLev C,
                                                    double* __restrict__ fc, double* __restrict__ uc, int kz) {
    const uint3 bk = xcd_block();
    const int nx = C.n[0] + 1, ny = C.n[1] + 1;
    const int t = bk.x * kNB + threadIdx.x;
    if (t >= nx * ny) return;
    const int I = t % nx, J = t / nx;
    const int K0 = bk.y * kz, K1 = min(K0 + kz - 1, C.n[2]);
    for (int K = K0; K <= K1; ++K) {
        const long long q = nidx(C, I, J, K);
        fc[q] = unknown(C, I, J, K) ? weighted(F, r, I, J, K) : 0.0;
        uc[q] = 0.0;
    }
}

// P e at fine node 2I + o: the mean of the coarse nodes I + o' (o' <= o),
// summed z, y, x
__device__ __forceinline__ double interpolated(const NLev& C, const double* e, int i, int j, int k) {
    const int I[3] = {i >> 1, j >> 1, k >> 1}, o[3] = {i & 1, j & 1, k & 1};
    double s = 0.0;
    for (int cz = 0; cz <= o[2]; ++cz)
        for (int cy = 0; cy <= o[1]; ++cy)
            for (int cx = 0; cx <= o[0]; ++cx)
                s = s + e[nidx(C, wrap(C, 0, I[0] + cx), wrap(C, 1, I[1] + cy), wrap(C, 2, I[2] + cz))];
    return s * (1.0 / (double)(1 << (o[0] + o[1] + o[2])));  // (a power of two: the quotient's bits)
}

// u_f += P e at the fine unknowns of the colours from c0 on (with sweeps after
// it colour 1 only: the first of them replaces colour 0 without reading it).
// Threads take the sweeps' positions: of a row's nodes of one colour all have
// the same parities, so a wave's lanes mostly sum the same 1, 2, 4 or 8 coarse
// nodes.  256^3: 69 us, against 159 a thread per node of both colours.
__global__ void __launch_bounds__(kNB) k_nd_prolong(NLev C, const double* __restrict__ e, NLev F,
                                                   double* __restrict__ u, int c0, int kz) {
    const uint3 bk = xcd_block();
    const int hx = (F.n[0] + 2) / 2, ny = F.n[1] + 1;
    const int t = bk.x * kNB + threadIdx.x;
    if (t >= hx * ny) return;
    const int tx = t % hx, j = t / hx;
    const int k0 = bk.y * kz, k1 = min(k0 + kz - 1, F.n[2]);
    for (int k = k0; k <= k1; ++k)
        for (int c = c0; c < 2; ++c) {
            const int i = 2 * tx + ((c - j - k) & 1);
            if (i > F.n[0] || !unknown(F, i, j, k)) continue;
            const long long q = nidx(F, i, j, k);
            u[q] = u[q] + interpolated(C, e, i, j, k);
        }
}

// the periodic copies n_d take the values of their nodes 0
__global__ void __launch_bounds__(kNB) k_nd_copies(NLev L, double* __restrict__ u) {
    for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < L.size;
         g += (long long)gridDim.x * blockDim.x) {
        int c[3];
        coords(L, g, c[0], c[1], c[2]);
        const long long q = nidx(L, c[0], c[1], c[2]);
        bool copy = false;
        for (int d = 0; d < 3; ++d)
            if (L.per[d] && c[d] == L.n[d]) { c[d] = 0; copy = true; }
        if (copy) u[q] = u[nidx(L, c[0], c[1], c[2])];
    }
}

// u -= mean over the unknowns, two passes: the sum (fixed per-block order,
// then block 0 adds the block sums in order), then the subtraction
__global__ void __launch_bounds__(kNB) k_nd_sum(NLev L, const double* __restrict__ u, double* __restrict__ part) {
    __shared__ double sh[2 * (kNB / 64)];
    double s = 0.0, c = 0.0;
    for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < L.size;
         g += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(L, g, i, j, k);
        if (unknown(L, i, j, k)) { s = s + u[nidx(L, i, j, k)]; c = c + 1.0; }
    }
    block_sum2(s, c, sh);
    if (threadIdx.x == 0) { part[2 * blockIdx.x] = s; part[2 * blockIdx.x + 1] = c; }
}
__global__ void __launch_bounds__(kNB) k_nd_sub(NLev L, double* __restrict__ u, const double* __restrict__ part,
                                               int nparts) {
    double s = 0.0, c = 0.0;
    for (int b = 0; b < nparts; ++b) { s = s + part[2 * b]; c = c + part[2 * b + 1]; }
    const double m = s / c;
    for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < L.size;
         g += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(L, g, i, j, k);
        if (unknown(L, i, j, k)) {
            const long long q = nidx(L, i, j, k);
            u[q] = u[q] - m;
        }
    }
}

// Bottom: FP64 CG on the unknowns in one workgroup (vectors in device memory
// or LDS, colour-split like the levels); fully periodic: right-hand side and
// solution projected to mean 0.  rtol on the L2 norm, at most 4 N iterations.
constexpr int kNBot = 1024;
__device__ __forceinline__ void nd_bottom(const NLev& L, double* x, const double* f, double* r, double* p, double* q,
                                          double rtol, int* iters, double* sh, double* bc) {
    const long long N = L.size;
    const bool sing = L.per[0] && L.per[1] && L.per[2];
    const double ih2 = 1.0 / (L.h * L.h);
    // sum over unknowns of a*b (or of a, with b == nullptr), broadcast
    auto dot = [&](const double* a, const double* b, double& cnt) {
        double s = 0.0, c = 0.0;
        for (long long g = threadIdx.x; g < N; g += blockDim.x) {
            int i, j, k;
            coords(L, g, i, j, k);
            if (!unknown(L, i, j, k)) continue;
            const long long o = nidx(L, i, j, k);
            s = s + (b ? a[o] * b[o] : a[o]);
            c = c + 1.0;
        }
        block_sum2(s, c, sh);
        if (threadIdx.x == 0) { bc[0] = s; bc[1] = c; }
        __syncthreads();
        cnt = bc[1];
        const double v = bc[0];
        __syncthreads();
        return v;
    };
    for (long long g = threadIdx.x; g < N; g += blockDim.x) {
        int i, j, k;
        coords(L, g, i, j, k);
        const long long o = nidx(L, i, j, k);
        r[o] = unknown(L, i, j, k) ? f[o] : 0.0;
        x[o] = 0.0;
    }
    __syncthreads();
    double cnt;
    if (sing) {
        const double m = dot(r, nullptr, cnt) / cnt;
        for (long long g = threadIdx.x; g < N; g += blockDim.x) {
            int i, j, k;
            coords(L, g, i, j, k);
            if (unknown(L, i, j, k)) {
                const long long o = nidx(L, i, j, k);
                r[o] = r[o] - m;
            }
        }
        __syncthreads();
    }
    for (long long g = threadIdx.x; g < N; g += blockDim.x) {
        int i, j, k;
        coords(L, g, i, j, k);
        const long long o = nidx(L, i, j, k);
        p[o] = r[o];
    }
    __syncthreads();
    double rs = dot(r, r, cnt);
    const double rs0 = rs;
    int it = 0;
    const long long maxit = 4 * (long long)cnt;
    if (rs0 != 0.0) {
        while (it < maxit) {
            for (long long g = threadIdx.x; g < N; g += blockDim.x) {
                int i, j, k;
                coords(L, g, i, j, k);
                const long long o = nidx(L, i, j, k);
                q[o] = unknown(L, i, j, k) ? (nsum(L, p, i, j, k) - 6.0 * p[o]) * ih2 : 0.0;
            }
            __syncthreads();
            const double alpha = rs / dot(p, q, cnt);
            for (long long g = threadIdx.x; g < N; g += blockDim.x) {
                int i, j, k;
                coords(L, g, i, j, k);
                if (!unknown(L, i, j, k)) continue;
                const long long o = nidx(L, i, j, k);
                x[o] = x[o] + alpha * p[o];
                r[o] = r[o] - alpha * q[o];
            }
            __syncthreads();
            const double rsn = dot(r, r, cnt);
            ++it;
            if (sqrt(rsn) <= rtol * sqrt(rs0)) break;
            const double beta = rsn / rs;
            for (long long g = threadIdx.x; g < N; g += blockDim.x) {
                int i, j, k;
                coords(L, g, i, j, k);
                if (unknown(L, i, j, k)) {
                    const long long o = nidx(L, i, j, k);
                    p[o] = r[o] + beta * p[o];
                }
            }
            __syncthreads();
            rs = rsn;
        }
        if (sing) {
            const double m = dot(x, nullptr, cnt) / cnt;
            for (long long g = threadIdx.x; g < N; g += blockDim.x) {
                int i, j, k;
                coords(L, g, i, j, k);
                if (unknown(L, i, j, k)) {
                    const long long o = nidx(L, i, j, k);
                    x[o] = x[o] - m;
                }
            }
        }
    }
    if (threadIdx.x == 0 && iters) *iters = it;
}
__global__ void __launch_bounds__(kNBot) k_nd_bottom(NLev L, double* __restrict__ x, const double* __restrict__ f,
                                                    double* __restrict__ r, double* __restrict__ p,
                                                    double* __restrict__ q, double rtol, int* __restrict__ iters) {
    __shared__ double sh[2 * (kNBot / 64)];
    __shared__ double bc[2];
    nd_bottom(L, x, f, r, p, q, rtol, iters, sh, bc);
}

// The V-cycle from a small level down in one workgroup, every level's u, f and
// r in LDS: f of the top level is read from device memory, its correction
// written there.  One launch per phase, each of a few blocks, is bound by
// launch and memory latency (3 to 6 us each, 11 phases a level); here a phase
// is a barrier and a few LDS round trips.  Same stages, node by node in the
// same arithmetic.  16^3 down to 2^3: 67 us a cycle against 120 in 34 launches.
constexpr int kNCoarse = 8;  // levels (each halves every direction)
struct NCoarse {
    NLev L[kNCoarse];
    int u[kNCoarse], f[kNCoarse], r[kNCoarse];  // offsets in LDS (elements)
    int bp, bq;
    int nl, nu1, nu2;
    double rtol;
};
__global__ void __launch_bounds__(kNBot) k_nd_coarse(NCoarse C, const double* __restrict__ ftop,
                                                    double* __restrict__ utop, int* __restrict__ iters) {
    extern __shared__ double sm[];
    __shared__ double sh[2 * (kNBot / 64)];
    __shared__ double bc[2];
    const int tid = threadIdx.x;
    // the nodes of one colour (rows of half slots)
    auto each = [&](const NLev& L, auto fn) {
        const unsigned hx = L.H, ny = L.n[1] + 1, rows = ny * (L.n[2] + 1), n = hx * rows;
        for (unsigned g = tid; g < n; g += kNBot) {
            const unsigned row = g / hx, k = row / ny;
            fn((int)g, (int)(g - row * hx), (int)(row - k * ny), (int)k);
        }
    };
    const Recip<double> r6(6.0);
    // a colour row's slot g is its offset in the colour block: neighbours are at
    // fixed distances, but through a periodic face
    auto sum6 = [&](const NLev& L, const double* u, int c, int g, int i, int j, int k) {
        const int H = L.H, P = H * (L.n[1] + 1), par = i & 1;
        const double* o = u + (1 - c) * (int)L.cs + g;
        const int xm = i == 0 ? L.n[0] / 2 - 1 : par - 1, xp = i == L.n[0] - 1 && L.per[0] ? -(i >> 1) : par;
        const int ym = j == 0 ? (L.n[1] - 1) * H : -H, yp = j == L.n[1] - 1 && L.per[1] ? -j * H : H;
        const int zm = k == 0 ? (L.n[2] - 1) * P : -P, zp = k == L.n[2] - 1 && L.per[2] ? -k * P : P;
        return ((o[xm] + o[xp]) + (o[ym] + o[yp])) + (o[zm] + o[zp]);
    };
    auto smooth = [&](const NLev& L, double* u, const double* f, int sweeps) {
        const double h2 = L.h * L.h;
        for (int c = 0; c < 2 * sweeps; ++c) {
            each(L, [&](int g, int t, int j, int k) {
                const int cc = c & 1, i = 2 * t + ((cc - j - k) & 1);
                if (i > L.n[0] || !unknown(L, i, j, k)) return;
                const int q = cc * (int)L.cs + g;
                u[q] = r6.div(sum6(L, u, cc, g, i, j, k) - h2 * f[q]);
            });
            __syncthreads();
        }
    };
    for (int q = tid; q < (int)C.L[0].alloc; q += kNBot) {
        sm[C.f[0] + q] = ftop[q];
        sm[C.u[0] + q] = 0.0;
    }
    __syncthreads();
    for (int l = 0; l + 1 < C.nl; ++l) {
        const NLev &L = C.L[l], &M = C.L[l + 1];
        double *u = sm + C.u[l], *f = sm + C.f[l], *r = sm + C.r[l], *fc = sm + C.f[l + 1], *uc = sm + C.u[l + 1];
        smooth(L, u, f, C.nu1);
        const double ih2 = 1.0 / (L.h * L.h);
        for (int c = 0; c < 2; ++c)
            each(L, [&](int g, int t, int j, int k) {
                const int i = 2 * t + ((c - j - k) & 1);
                if (i > L.n[0]) return;
                const int q = c * (int)L.cs + g;
                r[q] = unknown(L, i, j, k) ? f[q] - (sum6(L, u, c, g, i, j, k) - 6.0 * u[q]) * ih2 : 0.0;
            });
        __syncthreads();
        for (int c = 0; c < 2; ++c)
            each(M, [&](int, int t, int J, int K) {
                const int I = 2 * t + ((c - J - K) & 1);
                if (I > M.n[0]) return;
                const long long q = nidx(M, I, J, K);
                fc[q] = unknown(M, I, J, K) ? weighted(L, r, I, J, K) : 0.0;
                uc[q] = 0.0;
            });
        __syncthreads();
    }
    const int b = C.nl - 1;
    nd_bottom(C.L[b], sm + C.u[b], sm + C.f[b], sm + C.r[b], sm + C.bp, sm + C.bq, C.rtol, iters, sh, bc);
    __syncthreads();
    for (int l = C.nl - 2; l >= 0; --l) {
        const NLev &L = C.L[l], &M = C.L[l + 1];
        double *u = sm + C.u[l], *e = sm + C.u[l + 1];
        for (int c = C.nu2 > 0 ? 1 : 0; c < 2; ++c)
            each(L, [&](int, int t, int j, int k) {
                const int i = 2 * t + ((c - j - k) & 1);
                if (i > L.n[0] || !unknown(L, i, j, k)) return;
                const long long q = nidx(L, i, j, k);
                u[q] = u[q] + interpolated(M, e, i, j, k);
            });
        __syncthreads();
        smooth(L, u, sm + C.f[l], C.nu2);
    }
    for (int q = tid; q < (int)C.L[0].alloc; q += kNBot) utop[q] = sm[C.u[0] + q];
}

// Caller F-order node array <-> colour-split level array.
template <bool TO_SPLIT>
__global__ void __launch_bounds__(kNB) k_nd_convert(NLev L, double* __restrict__ fo, double* __restrict__ sp) {
    for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < L.size;
         g += (long long)gridDim.x * blockDim.x) {
        int i, j, k;
        coords(L, g, i, j, k);
        if constexpr (TO_SPLIT) sp[nidx(L, i, j, k)] = fo[g];
        else fo[g] = sp[nidx(L, i, j, k)];
    }
}

inline unsigned nblocks(long long n) { return (unsigned)std::min<long long>((n + kNB - 1) / kNB, 8192); }

// Planes each thread walks on a level: up to kmax, fewer where the level
// would otherwise give fewer than 2048 blocks.
inline int plane_depth(const NLev& L, bool half, int kmax) {
    const long long row = half ? (L.n[0] + 2) / 2 : L.n[0] + 1;
    const long long gx = (row * (L.n[1] + 1) + kNB - 1) / kNB;
    const long long kz = (gx * (L.n[2] + 1)) / 2048;
    return (int)std::max(1LL, std::min<long long>(kmax, kz));
}
// grid of the plane-walking kernels over the nodes of a level (half rows
// for the sweeps), kz planes per thread
inline dim3 plane_grid(const NLev& L, bool half, int kz) {
    const long long row = half ? (L.n[0] + 2) / 2 : L.n[0] + 1;
    return dim3((unsigned)((row * (L.n[1] + 1) + kNB - 1) / kNB), (unsigned)((L.n[2] + 1 + kz - 1) / kz), 1);
}
inline int plane_blocks(const NLev& L, bool half, int kz) {
    const dim3 g = plane_grid(L, half, kz);
    return (int)(g.x * g.y);
}
constexpr int kKZr = kKZ;  // residual
constexpr int kKZt = 2;    // transfers

// The nodal hierarchy of one geometry, cached on the context.
struct NHier {
    std::vector<NLev> L;
    std::vector<DevBuf<double>> u, f, r;
    DevBuf<double> part, bp, bq, fn;
    DevBuf<int> iters;
    std::string key;
    // streamed levels: their second iterate array, the sweeps before (level 0:
    // from its iterate, below from zero) and after the coarse levels
    std::vector<DevBuf<double>> a;
    std::vector<NSweep> pre, post;
    int coarse = -1;      // first level of the one-workgroup cycle (-1: none)
    NCoarse cc{};         // its levels
    size_t coarse_lds = 0;
};

// The levels of the one-workgroup cycle: as many as fit its LDS.
static void plan_coarse(NHier& H) {
    const int nl = (int)H.L.size();
    long long used = 2 * H.L[nl - 1].alloc;
    int first = nl;
    for (int l = nl - 1; l >= 1 && nl - l <= kNCoarse; --l) {
        used += 3 * H.L[l].alloc;
        if (used * 8 > lds_limit_bytes() - 1024) break;  // (1 KB: the kernel's own)
        first = l;
    }
    if (first >= nl - 1) return;
    NCoarse& C = H.cc;
    int at = 0;
    auto take = [&](long long n) {
        const int o = at;
        at += (int)n;
        return o;
    };
    C.nl = nl - first;
    for (int m = 0; m < C.nl; ++m) {
        C.L[m] = H.L[first + m];
        C.u[m] = take(C.L[m].alloc);
        C.f[m] = take(C.L[m].alloc);
        C.r[m] = take(C.L[m].alloc);
    }
    C.bp = take(H.L[nl - 1].alloc);
    C.bq = take(H.L[nl - 1].alloc);
    H.coarse = first;
    H.coarse_lds = (size_t)at * 8;
}

struct NCache {
    std::vector<std::unique_ptr<NHier>> h;  // most recent last
};

static NHier* get(bxmg_ctx ctx, const bxmg_ba_s* ba, double h0) {
    if (!ctx->nodal) ctx->nodal = std::make_shared<NCache>();
    NCache& C = *std::static_pointer_cast<NCache>(ctx->nodal);
    std::string key;
    auto put = [&](long long v) { key.append((const char*)&v, sizeof v); };
    long long hb;
    std::memcpy(&hb, &h0, sizeof hb);
    put(hb);
    for (int d = 0; d < 3; ++d) { put(ba->dom.n(d)); put(ba->per[d]); }
    for (size_t q = 0; q < C.h.size(); ++q)
        if (C.h[q]->key == key) return C.h[q].get();
    auto H = std::make_unique<NHier>();
    H->key = key;
    NLev l;
    for (int d = 0; d < 3; ++d) { l.n[d] = ba->dom.n(d); l.per[d] = ba->per[d]; }
    l.h = h0;
    for (;;) {
        l.size = (long long)(l.n[0] + 1) * (l.n[1] + 1) * (l.n[2] + 1);
        l.H = (l.n[0] + 2) / 2;
        l.cs = ((long long)l.H * (l.n[1] + 1) * (l.n[2] + 1) + 63) / 64 * 64;
        l.alloc = 2 * l.cs;
        H->L.push_back(l);
        bool more = true;
        for (int d = 0; d < 3; ++d)
            if (l.n[d] % 2 || l.n[d] <= 2) more = false;
        if (!more) break;
        for (int d = 0; d < 3; ++d) l.n[d] /= 2;
        l.h *= 2.0;
    }
    const NLev& B = H->L.back();
    if (B.size > 4096 * 8) throw std::runtime_error("nodal: bottom level too large");
    if (H->L[0].alloc >= (1LL << 31)) throw std::runtime_error("nodal: more than 2^31 nodes");
    const size_t nl = H->L.size();
    H->u.resize(nl);
    H->f.resize(nl);
    H->r.resize(nl);
    for (size_t q = 0; q < nl; ++q) {
        H->u[q].alloc(H->L[q].alloc);
        H->f[q].alloc(H->L[q].alloc);
        H->r[q].alloc(H->L[q].alloc);
    }
    plan_coarse(*H);
    const size_t end = H->coarse > 0 ? (size_t)H->coarse : nl - 1;
    int np = 8192;
    H->a.resize(nl);
    H->pre.resize(nl);
    H->post.resize(nl);
    for (size_t q = 0; q < end; ++q) {
        H->pre[q] = plan_nd_sweep(H->L[q], H->L[q + 1], q > 0, 1, false);
        H->post[q] = plan_nd_sweep(H->L[q], H->L[q + 1], false, q > 0 ? 0 : 2, true);
        np = std::max(np, H->post[q].blocks);
    }
    for (const NLev& l : H->L) np = std::max(np, plane_blocks(l, true, plane_depth(l, true, kKZr)));
    H->part.alloc(3 * (size_t)np);
    H->bp.alloc(B.alloc);
    H->bq.alloc(B.alloc);
    H->fn.alloc(3);
    H->iters.alloc(1);
    // last: a level whose second array finds no room is not streamed
    for (size_t q = 0; q < end; ++q) {
        if (!H->pre[q].nt) continue;
        try {
            H->a[q].alloc(H->L[q].alloc);
        } catch (HipError& e) {
            if (e.e != hipErrorOutOfMemory) throw;
            (void)hipGetLastError();
            H->pre[q].nt = 0;
        }
    }
    if (C.h.size() >= 4) C.h.erase(C.h.begin());
    C.h.push_back(std::move(H));
    return C.h.back().get();
}

// Returns the number of partial norms of its residual that the cycle left in
// H.part (0: none).
static int vcycle(NHier& H, size_t l, hipStream_t s, int nu1, int nu2, double brtol) {
    const NLev& L = H.L[l];
    if ((int)l == H.coarse) {
        static const hipError_t once = hipFuncSetAttribute(
            (const void*)k_nd_coarse, hipFuncAttributeMaxDynamicSharedMemorySize, lds_limit_bytes() - 1024);
        HIPCHK(once);
        NCoarse C = H.cc;
        C.nu1 = nu1;
        C.nu2 = nu2;
        C.rtol = brtol;
        hipLaunchKernelGGL(k_nd_coarse, dim3(1), dim3(kNBot), H.coarse_lds, s, C, H.f[l].p, H.u[l].p, H.iters.p);
        HIPCHK(hipGetLastError());
        return 0;
    }
    if (l + 1 == H.L.size()) {
        hipLaunchKernelGGL(k_nd_bottom, dim3(1), dim3(kNBot), 0, s, L, H.u[l].p, H.f[l].p, H.r[l].p, H.bp.p, H.bq.p,
                           brtol, H.iters.p);
        HIPCHK(hipGetLastError());
        return 0;
    }
    const int kg = plane_depth(L, true, kKZ), kr = plane_depth(L, true, kKZr);
    const dim3 gb = plane_grid(L, true, kg);
    const bool stream = nu1 == 2 && nu2 == 2 && H.pre[l].nt > 0;
    double* const u = stream ? H.a[l].p : H.u[l].p;
    if (stream) {
        if (l > 0)
            HIPCHK((launch_nd_sweep<true, 1, false>(s, L, H.pre[l], nullptr, u, H.f[l].p, H.r[l].p, nullptr, nullptr)));
        else
            HIPCHK((launch_nd_sweep<false, 1, false>(s, L, H.pre[l], H.u[l].p, u, H.f[l].p, H.r[l].p, nullptr,
                                                     nullptr)));
    } else {
        for (int q = 0; q < nu1; ++q)
            for (int c = 0; c < 2; ++c)
                hipLaunchKernelGGL(k_nd_gs, gb, dim3(kNB), 0, s, L, u, H.f[l].p, c, kg);
        hipLaunchKernelGGL(k_nd_resid, plane_grid(L, true, kr), dim3(kNB), 0, s, L, u, H.f[l].p, H.r[l].p, H.part.p,
                           kr);
    }
    const NLev& C = H.L[l + 1];
    const int kc = plane_depth(C, false, kKZt);
    hipLaunchKernelGGL(k_nd_restrict, plane_grid(C, false, kc), dim3(kNB), 0, s, L, H.r[l].p, C, H.f[l + 1].p,
                       H.u[l + 1].p, kc);
    vcycle(H, l + 1, s, nu1, nu2, brtol);
    if (stream) {
        double* const e = H.u[l + 1].p;
        if (l > 0)
            HIPCHK((launch_nd_sweep<false, 0, true>(s, L, H.post[l], u, H.u[l].p, H.f[l].p, nullptr, nullptr, e)));
        else
            HIPCHK((launch_nd_sweep<false, 2, true>(s, L, H.post[l], u, H.u[l].p, H.f[l].p, nullptr, H.part.p, e)));
        return l > 0 ? 0 : H.post[l].blocks;
    }
    hipLaunchKernelGGL(k_nd_prolong, gb, dim3(kNB), 0, s, C, H.u[l + 1].p, L, u, nu2 > 0 ? 1 : 0, kg);
    for (int q = 0; q < nu2; ++q)
        for (int c = 0; c < 2; ++c)
            hipLaunchKernelGGL(k_nd_gs, gb, dim3(kNB), 0, s, L, H.u[l].p, H.f[l].p, c, kg);
    HIPCHK(hipGetLastError());
    return 0;
}

}  // namespace nodal
}  // namespace bxmg

using namespace bxmg;

extern "C" bxmg_status bxmg_nodal_solve(bxmg_ctx ctx, const bxmg_solve_params* params, bxmg_boxarray ba,
                                        double* phi, const double* rhs, bxmg_solve_info* info) {
    if (!ctx || !ba || !phi || !rhs || !info) return fail(BXMG_EINVAL, "nodal_solve: NULL argument");
    std::memset(info, 0, sizeof(*info));
    bxmg_solve_params P;
    if (params) P = *params;
    else bxmg_solve_params_default(&P);
    if (P.nu1 < 0 || P.nu2 < 0 || P.max_cycles < 0 || P.precision != 0 || P.krylov != 0 || P.alpha != 0.0) {
        info->status = fail(BXMG_EINVAL, "nodal_solve: FP64 V-cycles of the Poisson operator only "
                                         "(precision 0, krylov 0, alpha 0)");
        return (bxmg_status)info->status;
    }
    const double h = (P.dx > 0) ? P.dx : 1.0 / ba->dom.n(0);
    std::lock_guard<std::mutex> lock(ctx->mu);
    const auto t0 = std::chrono::steady_clock::now();
    try {
        HIPCHK(hipSetDevice(ctx->device));
        nodal::NHier* H = nodal::get(ctx, ba, h);
        const hipStream_t s = ctx->stream;
        const nodal::NLev& L0 = H->L[0];
        info->levels = (int)H->L.size();
        const unsigned nb = nodal::nblocks(L0.size);
        // the caller's arrays into the colour-split level arrays
        HIPCHK(hipMemsetAsync(H->u[0].p, 0, L0.alloc * sizeof(double), s));
        HIPCHK(hipMemsetAsync(H->f[0].p, 0, L0.alloc * sizeof(double), s));
        hipLaunchKernelGGL(nodal::k_nd_convert<true>, dim3(nb), dim3(nodal::kNB), 0, s, L0, phi, H->u[0].p);
        hipLaunchKernelGGL(nodal::k_nd_convert<true>, dim3(nb), dim3(nodal::kNB), 0, s, L0, (double*)rhs, H->f[0].p);
        HIPCHK(hipGetLastError());
        const int kr0 = nodal::plane_depth(L0, true, nodal::kKZr);
        // norms reduced on the device and read back: of f (fonly) or of the
        // residual of the current iterate, unless taken partials hold it
        auto norms = [&](bool fonly, int taken, double out[3]) {
            if (taken) {
            } else if (fonly)
                hipLaunchKernelGGL(nodal::k_nd_fnorm, dim3(nb), dim3(nodal::kNB), 0, s, L0, H->f[0].p, H->part.p);
            else
                hipLaunchKernelGGL(nodal::k_nd_resid, nodal::plane_grid(L0, true, kr0), dim3(nodal::kNB), 0, s, L0,
                                   H->u[0].p, H->f[0].p, H->r[0].p, H->part.p, kr0);
            HIPCHK(hipGetLastError());
            HIPCHK(launch_norm_final(s, H->part.p, taken ? taken : fonly ? (int)nb : nodal::plane_blocks(L0, true, kr0),
                                     H->fn.p));
            HIPCHK(hipMemcpyAsync(ctx->h_norm, H->fn.p, 3 * sizeof(double), hipMemcpyDeviceToHost, s));
            HIPCHK(hipStreamSynchronize(s));
            out[0] = ctx->h_norm[2] > 0.0 ? (double)NAN : ctx->h_norm[0];
            out[1] = ctx->h_norm[1];
            out[2] = ctx->h_norm[2];
        };
        double fz[3];
        norms(true, 0, fz);
        const double fnorm = fz[0];
        info->f_inf = fnorm;
        int status = 0, cyc = 0;
        if (!(fnorm == fnorm)) {
            status = BXMG_ENONFINITE;
        } else if (fnorm > 0.0) {
            for (int taken = 0;; ++cyc) {
                double rn[3];
                norms(false, taken, rn);
                if (cyc < kHist) {
                    info->hist[cyc] = rn[0] / fnorm;
                    info->hist_l2[cyc] = std::sqrt(rn[1]);
                    info->nhist = cyc + 1;
                }
                info->rel_resid_inf = rn[0] / fnorm;
                info->resid_l2 = std::sqrt(rn[1]);
                if (!(rn[0] == rn[0])) { status = BXMG_ENONFINITE; break; }
                if (P.fixed_cycles > 0) {
                    if (cyc == P.fixed_cycles) break;
                } else {
                    if (rn[0] <= P.rel_tol * fnorm || rn[0] <= P.abs_tol) break;
                    if (cyc == P.max_cycles) { status = BXMG_ENOCONV; break; }
                }
                taken = nodal::vcycle(*H, 0, s, P.nu1, P.nu2, P.bottom_rtol);
            }
        } else {
            HIPCHK(hipMemsetAsync(H->u[0].p, 0, L0.alloc * sizeof(double), s));  // f == 0: u = 0
        }
        info->cycles = cyc;
        if (status == 0) {
            if (L0.per[0] && L0.per[1] && L0.per[2]) {
                hipLaunchKernelGGL(nodal::k_nd_sum, dim3(nb), dim3(nodal::kNB), 0, s, L0, H->u[0].p, H->part.p);
                hipLaunchKernelGGL(nodal::k_nd_sub, dim3(nb), dim3(nodal::kNB), 0, s, L0, H->u[0].p, H->part.p,
                                   (int)nb);
            }
            hipLaunchKernelGGL(nodal::k_nd_copies, dim3(nodal::nblocks(L0.size)), dim3(nodal::kNB), 0, s, L0,
                               H->u[0].p);
            HIPCHK(hipGetLastError());
            hipLaunchKernelGGL(nodal::k_nd_convert<false>, dim3(nb), dim3(nodal::kNB), 0, s, L0, phi, H->u[0].p);
            HIPCHK(hipGetLastError());
        }
        HIPCHK(hipStreamSynchronize(s));
        info->status = status;
        if (status == BXMG_ENOCONV) fail(BXMG_ENOCONV, "nodal_solve: max_cycles reached");
        if (status == BXMG_ENONFINITE) fail(BXMG_ENONFINITE, "nodal_solve: non-finite values");
    } catch (HipError& e) {
        info->status = fail(BXMG_EDEVICE, std::string("nodal_solve: ") + e.where + ": " + hipGetErrorString(e.e));
    } catch (std::exception& e) {
        info->status = fail(BXMG_EINVAL, std::string("nodal_solve: ") + e.what());
    }
    info->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return (bxmg_status)info->status;
}
