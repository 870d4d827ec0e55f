// The fused coarse V-cycle: every level below the first of at most
// kMaxBottomCells cells, down to the conjugate-gradient bottom and back, by
// one workgroup per problem in one launch.
//
// These levels are all latency: a 16^3 level is 2048 x-pairs, 8^3 is 256.  A
// thread holds its pairs' cells (both colours), right-hand side and operator
// coefficients in registers -- four pairs of the top level, one of every
// level below -- and the levels' u lies in LDS, colour by colour, without
// ghost cells: a neighbour beyond a Dirichlet face is the cell itself with
// its sign turned (its value before the update, as a ghost refreshed after
// each half-sweep holds), one across a periodic face the wrapped cell.  So a
// half-sweep is five LDS reads, about a dozen instructions and one barrier
// per cell; levels of at most 64 pairs run in one wave without barriers, and
// so does the bottom.  Each cell's arithmetic and the order of its sums are
// those of the level-by-level kernels.
//
// Measured, per cycle, against levels with ghost cells in LDS and 1024
// threads (one cell per thread and step, indexes formed for every cell, ghost
// stores after each update, three barriers per sum of the bottom):
//   16^3 FP64 ... 2^3                      59 -> 24 us
//   12 x 6 x 10 FP64, bottom of 90 cells   98 -> 26 us
//   16^3 FP32, variable coefficient        72 -> 31 us
// What is left is the chain of about 40 barriers and CG steps, and the first
// fetch of 128 KB of code.
#include <hip/hip_runtime.h>
#include <type_traits>

#include "bxmg_device.h"

namespace bxmg {

namespace {

constexpr int kCT = 512;  // threads of the workgroup
constexpr int kTopPairs = kMaxBottomCells / 2 / kCT;

extern __shared__ __align__(16) unsigned char coarse_lds[];

// a pointer kept in the LDS copy of the descriptor, known to be to device
// memory (else its accesses would be flat ones)
template <class T>
using dev_ptr = __attribute__((address_space(1))) T*;
template <class T>
__device__ __forceinline__ dev_ptr<T> dev(T* p) { return (dev_ptr<T>)p; }

// orders LDS writes before later LDS reads of other threads: of one wave, or
// of the workgroup
template <bool WAVE>
__device__ __forceinline__ void lds_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
}

// a = q d + r for 0 <= a < 2^20, d >= 1: the float estimate is off by less
// than one, so one correction makes it exact
__device__ __forceinline__ void divmod20(int a, int d, int& q, int& r) {
    q = (int)((float)a * (1.0f / (float)d));
    r = a - q * d;
    if (r < 0) { --q; r += d; }
    else if (r >= d) { ++q; r -= d; }
}

// The LDS of one level: u as two half arrays of P pairs (colour 0, colour 1),
// f the same way.  The bottom's u is one array in natural order.
template <class T>
struct LevLds {
    int nx, ny, nz, P;
    T* u;
    T* f;
};

// value of cell (I, J, K) of a level's u with ghosts resolved by the caller
template <class T>
__device__ __forceinline__ T lev_u(const LevLds<T>& C, bool natural, int I, int J, int K) {
    const int row = J + C.ny * K;
    if (natural) return C.u[I + C.nx * row];
    return C.u[((I + J + K) & 1) * C.P + (I >> 1) + (C.nx >> 1) * row];
}

// KP x-pairs of a level per thread.
template <class T, int MODE, int KP>
struct Pairs {
    T u[KP][2], f[KP][2];      // by colour
    int nb[KP][2][5];          // element of the neighbours of the colour-c cell: x, y-, y+, z-, z+
    T w[KP][2][6];             // their weights (sign, or signed face coefficient); [5]: the pair's other cell
    T sb[KP][2];               // MODE 2: diagonal
    int t[KP], m[KP], y[KP], z[KP];
    bool on[KP];
    T h2, ih2, b;
    Recip<T> rec{T(1)};

    __device__ __forceinline__ void setup(const LevLds<T>& L, const CoarseGeom<T>& g, int l) {
        const double h = g.h[l], a = g.a;
        h2 = (T)(h * h);
        ih2 = (T)(1.0 / (h * h));
        const T dg = (T)(a * (h * h));
        b = T(6) + dg;
        if constexpr (MODE == 0) rec = Recip<T>(b);
        const int nm = L.nx >> 1;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            t[k] = (int)threadIdx.x + k * kCT;
            on[k] = t[k] < L.P;
            const int tt = on[k] ? t[k] : 0;
            int r;
            divmod20(tt, nm, r, m[k]);
            divmod20(r, L.ny, z[k], y[k]);
            const int my = m[k], yy = y[k], zz = z[k], sy = nm, sz = nm * L.ny;
            // neighbour pair of each direction, or -1 beyond a Dirichlet face
            const int xl = my > 0 ? tt - 1 : g.per[0] ? tt + nm - 1 : -1;
            const int xr = my < nm - 1 ? tt + 1 : g.per[0] ? tt - (nm - 1) : -1;
            const int yd = yy > 0 ? tt - sy : g.per[1] ? tt + (L.ny - 1) * sy : -1;
            const int yu = yy < L.ny - 1 ? tt + sy : g.per[1] ? tt - (L.ny - 1) * sy : -1;
            const int zd = zz > 0 ? tt - sz : g.per[2] ? tt + (L.nz - 1) * sz : -1;
            const int zu = zz < L.nz - 1 ? tt + sz : g.per[2] ? tt - (L.nz - 1) * sz : -1;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int o = (c + yy + zz) & 1;
                const int n5[5] = {o ? xr : xl, yd, yu, zd, zu};
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    nb[k][c][q] = n5[q] >= 0 ? (c ^ 1) * L.P + n5[q] : c * L.P + tt;
                    w[k][c][q] = n5[q] >= 0 ? T(1) : T(-1);
                }
                if constexpr (MODE == 2) {
                    const int x = 2 * my + o, nx = L.nx, ny = L.ny;
                    const int ix = x + (nx + 1) * (yy + ny * zz);
                    const int iy = x + nx * (yy + (ny + 1) * zz);
                    const int iz = x + nx * (yy + ny * zz);
                    const auto cx = dev(g.c[l][0]), cy = dev(g.c[l][1]), cz = dev(g.c[l][2]);
                    const T bxm = cx[ix], bxp = cx[ix + 1];
                    const T bym = cy[iy], byp = cy[iy + nx];
                    const T bzm = cz[iz], bzp = cz[iz + nx * ny];
                    sb[k][c] = (((bxm + bxp) + (bym + byp)) + (bzm + bzp)) + dg;
                    w[k][c][0] *= o ? bxp : bxm;
                    w[k][c][5] = o ? bxm : bxp;
                    w[k][c][1] *= bym;
                    w[k][c][2] *= byp;
                    w[k][c][3] *= bzm;
                    w[k][c][4] *= bzp;
                }
            }
        }
    }
    // su of the colour-c cell of pair k (x- + x+ commutes; a weight of +-1
    // multiplies exactly, so the fma rounds as the sum does)
    __device__ __forceinline__ T sum(const T* __restrict__ lu, int k, int c) const {
        const T xn = lu[nb[k][c][0]], yd = lu[nb[k][c][1]], yu = lu[nb[k][c][2]], zd = lu[nb[k][c][3]],
                zu = lu[nb[k][c][4]];
        const T o = u[k][c ^ 1];
        const T* W = w[k][c];
        if constexpr (MODE == 0)
            return (Recip<T>::fma_(W[0], xn, o) + Recip<T>::fma_(W[2], yu, W[1] * yd)) +
                   Recip<T>::fma_(W[4], zu, W[3] * zd);
        else
            return ((W[0] * xn + W[5] * o) + (W[1] * yd + W[2] * yu)) + (W[3] * zd + W[4] * zu);
    }
    template <bool WAVE>
    __device__ __forceinline__ void half_sweep(const LevLds<T>& L, int c, bool zero) {
        T v[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (!on[k]) continue;
            // u = 0: the neighbour sum is +0 and nothing is read
            const T su = zero ? T(0) : sum(L.u, k, c);
            const T rhs = su - h2 * f[k][c];
            if constexpr (MODE == 0) v[k] = rec.div(rhs);
            else v[k] = rhs / sb[k][c];
        }
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (!on[k]) continue;
            u[k][c] = v[k];
            L.u[c * L.P + t[k]] = v[k];
        }
        lds_sync<WAVE>();
    }
    template <bool WAVE>
    __device__ __forceinline__ void smooth(const LevLds<T>& L, int nsweeps) {
        for (int s = 0; s < nsweeps; ++s) {
            half_sweep<WAVE>(L, 0, false);
            half_sweep<WAVE>(L, 1, false);
        }
    }
    // pre-smoothing from u = 0; the level's f is in the registers
    template <bool WAVE>
    __device__ __forceinline__ void pre(const LevLds<T>& L, int nu1) {
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            u[k][0] = T(0);
            u[k][1] = T(0);
        }
        if (nu1 > 0) {
            half_sweep<WAVE>(L, 0, true);
            // colour 1 reads colour 0 and, beside a Dirichlet face, its own
            // old value: put it in place
#pragma unroll
            for (int k = 0; k < KP; ++k)
                if (on[k]) L.u[L.P + t[k]] = T(0);
            half_sweep<WAVE>(L, 1, false);
            smooth<WAVE>(L, nu1 - 1);
        } else {
#pragma unroll
            for (int k = 0; k < KP; ++k)
                if (on[k]) {
                    L.u[t[k]] = T(0);
                    L.u[L.P + t[k]] = T(0);
                }
            lds_sync<WAVE>();
        }
    }
    // the sum of the two residuals of every pair into S
    template <bool WAVE>
    __device__ __forceinline__ void resid(const LevLds<T>& L, T* __restrict__ S) const {
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (!on[k]) continue;
            T r[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const T su = sum(L.u, k, c);
                r[c] = f[k][c] - (su - (MODE == 0 ? b : sb[k][c]) * u[k][c]) * ih2;
            }
            S[t[k]] = r[0] + r[1];
        }
        lds_sync<WAVE>();
    }
    // u += P e (the coarse level C), then into LDS
    template <bool WAVE>
    __device__ __forceinline__ void prolong(const LevLds<T>& L, const LevLds<T>& C, bool natural, const int* per,
                                            int order) {
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (!on[k]) continue;
            const int I = m[k], J = y[k] >> 1, K = z[k] >> 1;
            T e[2];  // of the cells x = 2m, 2m + 1
            if (order == 1) {
                e[0] = e[1] = lev_u(C, natural, I, J, K);
            } else {
                // the neighbours on the children's sides; beyond a Dirichlet
                // face the cell itself with its sign turned
                auto side = [](int i, int d, int n, int p, int& j, T& s) {
                    j = i + d;
                    s = T(1);
                    if (j < 0) { j = p ? n - 1 : 0; s = p ? T(1) : T(-1); }
                    if (j >= n) { j = p ? 0 : n - 1; s = p ? T(1) : T(-1); }
                };
                int X[2], Jn, Kn;
                T sx[2], sj, sk;
                side(I, -1, C.nx, per[0], X[0], sx[0]);
                side(I, 1, C.nx, per[0], X[1], sx[1]);
                side(J, (y[k] & 1) ? 1 : -1, C.ny, per[1], Jn, sj);
                side(K, (z[k] & 1) ? 1 : -1, C.nz, per[2], Kn, sk);
                const T c000 = lev_u(C, natural, I, J, K), c010 = sj * lev_u(C, natural, I, Jn, K);
                const T c001 = sk * lev_u(C, natural, I, J, Kn), c011 = (sj * sk) * lev_u(C, natural, I, Jn, Kn);
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const T c100 = sx[o] * lev_u(C, natural, X[o], J, K);
                    const T c110 = (sx[o] * sj) * lev_u(C, natural, X[o], Jn, K);
                    const T c101 = (sx[o] * sk) * lev_u(C, natural, X[o], J, Kn);
                    const T c111 = (sx[o] * sj * sk) * lev_u(C, natural, X[o], Jn, Kn);
                    e[o] = (((T(27) * c000 + T(9) * ((c100 + c010) + c001)) + T(3) * ((c110 + c101) + c011)) + c111) *
                           T(0.015625);
                }
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int o = (c + y[k] + z[k]) & 1;
                u[k][c] = u[k][c] + (o ? e[1] : e[0]);
                L.u[c * L.P + t[k]] = u[k][c];
            }
        }
        lds_sync<WAVE>();
    }
};

// Coarse right-hand side at (I, J, K) from the fine level's pair sums.
template <class T>
__device__ __forceinline__ T restricted(const T* __restrict__ S, int fnm, int fny, int I, int J, int K) {
    const int p = I + fnm * (2 * J + fny * 2 * K), q = p + fnm * fny;
    return ((S[p] + S[p + fnm]) + (S[q] + S[q + fnm])) * T(0.125);
}

// Sum of K terms per thread over a wave or the workgroup, the same value in
// every thread and in the order of the one-wave and 1024-thread reductions of
// the stand-alone bottom solve: lanes in a butterfly, far partners first (the
// near ones by DPP), then 64 cells after 64 cells; beyond 1024 cells a lane
// first adds its cells 1024 apart.  lanes: only lanes below this power of two
// hold terms.  The workgroup's partial sums use two buffers in turn, so one
// barrier per sum is enough.
template <int K, bool WAVE>
struct Sum {
    double* sh;
    int turn = 0, lanes;
    __device__ Sum(double* s, int n) : sh(s), lanes(n) {}
    template <class F>
    static __device__ __forceinline__ double both(double v, F f) {  // f on the two halves
        const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
        const unsigned lo = f((int)(unsigned)b), hi = f((int)(unsigned)(b >> 32));
        return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
    }
    template <int C>
    static __device__ __forceinline__ double dpp(double v) {
        return both(v, [](int x) { return (unsigned)__builtin_amdgcn_mov_dpp(x, C, 0xf, 0xf, true); });
    }
    __device__ __forceinline__ double butterfly(double v) const {
        if (lanes > 32) v = v + __shfl_xor(v, 32);
        if (lanes > 16) v = v + __shfl_xor(v, 16);
        if (lanes > 8) v = v + dpp<0x128>(v);  // row_ror:8
        v = v + both(v, [](int x) { return (unsigned)__builtin_amdgcn_ds_swizzle(x, (4 << 10) | 0x1f); });  // xor 4
        v = v + dpp<0x4E>(v);  // quad_perm [2,3,0,1]
        v = v + dpp<0xB1>(v);  // quad_perm [1,0,3,2]
        return v;
    }
    template <class Term>
    __device__ __forceinline__ double operator()(Term term) {
        if constexpr (WAVE) {
            double v = butterfly(term(0));
#pragma unroll
            for (int k = 1; k < K; ++k) v = v + butterfly(term(k));
            return both(v, [](int x) { return (unsigned)__builtin_amdgcn_readfirstlane(x); });
        } else {
            constexpr int NV = K > 1 ? 2 : 1, NW = kCT / 64;  // the halves of 1024 cells
            double* s = sh + turn * 2 * NW;
            turn ^= 1;
#pragma unroll
            for (int e = 0; e < NV; ++e) {
                double v = 0.0;
#pragma unroll
                for (int k = e; k < K; k += NV) v = v + term(k);
                v = butterfly(v);
                if ((threadIdx.x & 63) == 0) s[e * NW + (threadIdx.x >> 6)] = v;
            }
            lds_sync<false>();
            double v = s[0];
            for (int w = 1; w < NV * NW; ++w) v = v + s[w];
            return v;
        }
    }
};

// FP64 conjugate gradients on the bottom: K cells per thread, of one wave or
// of the workgroup; fv(n) the right-hand side of cell n (natural order),
// put(n, x) its result.  p is N doubles of LDS.  The stop test and projection
// are those of the stand-alone bottom solve.
template <class T, int MODE, int K, bool WAVE, class FV, class Put>
__device__ __forceinline__ void bottom_owned(const CoarseGeom<T>& g, double* __restrict__ p, double* __restrict__ sh,
                                             FV fv, Put put) {
    constexpr int NT = WAVE ? 64 : kCT;
    constexpr bool kKeep = K <= 2;  // neighbours and coefficients kept in registers
    const int l = g.nlev - 1;
    const int nx = g.n[l][0], ny = g.n[l][1], nz = g.n[l][2], N = nx * ny * nz;
    const double h = g.h[l], ih2 = 1.0 / (h * h), dg = g.a * (h * h);
    const int tid = threadIdx.x;
    auto place = [&](int n, int* q, double* w) {
        int r, a, b, c;
        divmod20(n, nx, r, a);
        divmod20(r, ny, c, b);
        const int sy = nx, sz = nx * ny;
        const int d[6] = {a > 0 ? n - 1 : g.per[0] ? n + nx - 1 : -1, a < nx - 1 ? n + 1 : g.per[0] ? n - (nx - 1) : -1,
                          b > 0 ? n - sy : g.per[1] ? n + (ny - 1) * sy : -1,
                          b < ny - 1 ? n + sy : g.per[1] ? n - (ny - 1) * sy : -1,
                          c > 0 ? n - sz : g.per[2] ? n + (nz - 1) * sz : -1,
                          c < nz - 1 ? n + sz : g.per[2] ? n - (nz - 1) * sz : -1};
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            q[k] = d[k] >= 0 ? d[k] : n;
            w[k] = d[k] >= 0 ? 1.0 : -1.0;
        }
        double sb = 6.0;
        if constexpr (MODE == 2) {
            const int ix = a + (nx + 1) * (b + ny * c), iy = a + nx * (b + (ny + 1) * c), iz = n;
            const auto cx = dev(g.c[l][0]), cy = dev(g.c[l][1]), cz = dev(g.c[l][2]);
            const double bxm = (double)cx[ix], bxp = (double)cx[ix + 1];
            const double bym = (double)cy[iy], byp = (double)cy[iy + nx];
            const double bzm = (double)cz[iz], bzp = (double)cz[iz + nx * ny];
            sb = ((bxm + bxp) + (bym + byp)) + (bzm + bzp);
            w[0] *= bxm; w[1] *= bxp; w[2] *= bym; w[3] *= byp; w[4] *= bzm; w[5] *= bzp;
        }
        return sb + dg;
    };
    int q[kKeep ? K : 1][6];
    double w[kKeep ? K : 1][6], sb[kKeep ? K : 1];
    double r[K], x[K], pv[K], qv[K];
    bool on[K];
    int lanes = 64;
    if (WAVE && K == 1)
        while (lanes > 8 && lanes / 2 >= N) lanes /= 2;
    Sum<K, WAVE> sum(sh, lanes);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int n = tid + k * NT;
        on[k] = n < N;
        r[k] = on[k] ? fv(n) : 0.0;
        x[k] = 0.0;
        if constexpr (kKeep) sb[k] = place(on[k] ? n : 0, q[k], w[k]);
    }
    const bool sing = g.per[0] && g.per[1] && g.per[2] && g.a == 0.0;
    auto total = [&](auto term) { return sum([&](int k) { return on[k] ? term(k) : 0.0; }); };
    if (sing) {
        const double mean = total([&](int k) { return r[k]; }) / (double)N;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (on[k]) r[k] = r[k] - mean;
    }
    double rs = total([&](int k) { return r[k] * r[k]; });
    const double rs0 = rs;
    int it = 0;
    if (rs0 != 0.0) {
        const double stop = g.rtol * sqrt(rs0);
        const int maxit = 4 * N;
#pragma unroll
        for (int k = 0; k < K; ++k) pv[k] = r[k];
        while (it < maxit) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (on[k]) p[tid + k * NT] = pv[k];
            lds_sync<WAVE>();
#pragma unroll
            for (int k = 0; k < K; ++k) {
                qv[k] = 0.0;
                if (!on[k]) continue;
                int qq[6];
                double ww[6], s;
                if constexpr (kKeep) {
                    s = sb[k];
                    for (int d = 0; d < 6; ++d) { qq[d] = q[k][d]; ww[d] = w[k][d]; }
                } else {
                    s = place(tid + k * NT, qq, ww);
                }
                const double su = ((ww[0] * p[qq[0]] + ww[1] * p[qq[1]]) + (ww[2] * p[qq[2]] + ww[3] * p[qq[3]])) +
                                  (ww[4] * p[qq[4]] + ww[5] * p[qq[5]]);
                qv[k] = (su - s * pv[k]) * ih2;
            }
            // (its barrier also keeps this step's reads of p before the next writes)
            const double pAp = total([&](int k) { return pv[k] * qv[k]; });
            const double alpha = rs / pAp;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                x[k] = x[k] + alpha * pv[k];
                r[k] = r[k] - alpha * qv[k];
            }
            const double rsn = total([&](int k) { return r[k] * r[k]; });
            ++it;
            if (sqrt(rsn) <= stop) break;
            const double beta = rsn / rs;
#pragma unroll
            for (int k = 0; k < K; ++k) pv[k] = r[k] + beta * pv[k];
            rs = rsn;
            if constexpr (WAVE) lds_sync<true>();
        }
        if (sing) {
            const double mean = total([&](int k) { return x[k]; }) / (double)N;
#pragma unroll
            for (int k = 0; k < K; ++k) x[k] = x[k] - mean;
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (on[k]) put(tid + k * NT, x[k]);
    if (tid == 0 && g.iters) *dev(g.iters) = it;
}

}  // namespace

// LDS: per smoothed level u and f (2 P each), the top level's pair sums, the
// bottom's result (N, natural order), then the CG's p (N doubles) and sums.
template <class T, int MODE>
__global__ void __launch_bounds__(kCT) k_coarse_fast(const CoarseCycle<T>* __restrict__ ccs,
                                                    const int* __restrict__ active) {
    static_assert(sizeof(CoarseGeom<T>) % 4 == 0 && sizeof(CoarseGeom<T>) / 4 <= kCT, "descriptor copy");
    __shared__ CoarseGeom<T> g;
    {
        const int* src = (const int*)&ccs[blockIdx.x].g;
        if (threadIdx.x < sizeof(CoarseGeom<T>) / 4) ((int*)&g)[threadIdx.x] = src[threadIdx.x];
        __syncthreads();
    }
    if (active && !active[g.pid]) return;
    const int nl = g.nlev, bot = nl - 1;
    T* base = (T*)coarse_lds;
    auto level = [&](int l) {
        LevLds<T> L;
        T* at = base;
        for (int k = 0; k < l; ++k) at += 2 * g.n[k][0] * g.n[k][1] * g.n[k][2];
        L.nx = g.n[l][0];
        L.ny = g.n[l][1];
        L.nz = g.n[l][2];
        L.P = (L.nx >> 1) * L.ny * L.nz;
        L.u = at;
        L.f = at + 2 * L.P;
        return L;
    };
    // the bottom's u, after every smoothed level's arrays and the pair sums
    T* S = level(bot).u;
    const int N = g.n[bot][0] * g.n[bot][1] * g.n[bot][2];
    T* ub = S + (nl > 1 ? (g.n[0][0] >> 1) * g.n[0][1] * g.n[0][2] : 0);
    double* cg_p = (double*)(coarse_lds + ((((unsigned)(ub - base) + N) * sizeof(T) + 15) & ~15u));
    double* cg_sh = cg_p + N;
    LevLds<T> B;
    B.nx = g.n[bot][0];
    B.ny = g.n[bot][1];
    B.nz = g.n[bot][2];
    B.P = 0;
    B.u = ub;
    B.f = nullptr;

    const int tid = threadIdx.x;
    const auto gf = dev(g.f);
    const auto gu = dev(g.u);
    // element of cell (x, y, z) in the top level's storage
    auto top_elem = [&](int x, int y, int z) {
        return ((x + y + z + g.par) & 1) * g.cs + (z + 1) * g.GH + (y + 1) * g.H + ((x + 1) >> 1);
    };
    if (nl == 1) {  // the bottom alone, from and to device memory
        auto xyz = [&](int n) {
            int r, a, b, c;
            divmod20(n, B.nx, r, a);
            divmod20(r, B.ny, c, b);
            return top_elem(a, b, c);
        };
        auto fv = [&](int n) { return (double)gf[xyz(n)]; };
        auto put = [&](int n, double v) { gu[xyz(n)] = (T)v; };
        if (N <= 64) {
            if (tid < 64) bottom_owned<T, MODE, 1, true>(g, cg_p, cg_sh, fv, put);
        } else if (N <= 128) {
            if (tid < 64) bottom_owned<T, MODE, 2, true>(g, cg_p, cg_sh, fv, put);
        } else if (N <= kCT) {
            bottom_owned<T, MODE, 1, false>(g, cg_p, cg_sh, fv, put);
        } else {
            bottom_owned<T, MODE, kMaxBottomCells / kCT, false>(g, cg_p, cg_sh, fv, put);
        }
        return;
    }

    const LevLds<T> T0 = level(0);
    Pairs<T, MODE, kTopPairs> A;
    A.setup(T0, g, 0);
#pragma unroll
    for (int k = 0; k < kTopPairs; ++k)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int o = (c + A.y[k] + A.z[k]) & 1;
            A.f[k][c] = A.on[k] ? gf[top_elem(2 * A.m[k] + o, A.y[k], A.z[k])] : T(0);
        }
    A.template pre<false>(T0, g.nu1);
    A.template resid<false>(T0, S);

    // levels below, one pair per thread; from the first of at most 64 pairs
    // on they belong to wave 0 alone
    Pairs<T, MODE, 1> D;
    auto take_f = [&](const LevLds<T>& F, const LevLds<T>& C) {  // f of level C from F's pair sums
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int o = (c + D.y[0] + D.z[0]) & 1;
            D.f[0][c] = T(0);
            if (D.on[0]) {
                D.f[0][c] = restricted(S, F.nx >> 1, F.ny, 2 * D.m[0] + o, D.y[0], D.z[0]);
                C.f[c * C.P + D.t[0]] = D.f[0][c];
            }
        }
    };
    auto down = [&](int l, auto wave) {
        constexpr bool W = decltype(wave)::value;
        const LevLds<T> F = level(l - 1), C = level(l);
        D.setup(C, g, l);
        take_f(F, C);  // (pre-smoothing's barriers keep these reads before the next sums)
        D.template pre<W>(C, g.nu1);
        D.template resid<W>(C, S);
    };
    auto up = [&](int l, auto wave) {
        constexpr bool W = decltype(wave)::value;
        const LevLds<T> F = level(l);
        D.setup(F, g, l);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            D.f[0][c] = D.on[0] ? F.f[c * F.P + D.t[0]] : T(0);
            D.u[0][c] = D.on[0] ? F.u[c * F.P + D.t[0]] : T(0);
        }
        D.template prolong<W>(F, l + 1 == bot ? B : level(l + 1), l + 1 == bot, g.per, g.prolong);
        D.template smooth<W>(F, g.nu2);
    };
    auto bottom = [&](auto wave) {
        constexpr bool W = decltype(wave)::value;
        const LevLds<T> F = level(bot - 1);
        auto fv = [&](int n) {
            int r, a, b, c;
            divmod20(n, B.nx, r, a);
            divmod20(r, B.ny, c, b);
            return (double)restricted(S, F.nx >> 1, F.ny, a, b, c);
        };
        auto put = [&](int n, double v) { ub[n] = (T)v; };
        if constexpr (W) {
            if (N <= 64) bottom_owned<T, MODE, 1, true>(g, cg_p, cg_sh, fv, put);
            else bottom_owned<T, MODE, 2, true>(g, cg_p, cg_sh, fv, put);
        } else {
            bottom_owned<T, MODE, 1, false>(g, cg_p, cg_sh, fv, put);  // an eighth of at most 4096 cells
        }
        lds_sync<W>();
    };
    int lw = 1;
    while (lw < bot && (g.n[lw][0] >> 1) * g.n[lw][1] * g.n[lw][2] > 64) ++lw;
    for (int l = 1; l < lw; ++l) down(l, std::false_type());
    if (lw < bot || N <= 128) {
        if (tid < 64) {
            for (int l = lw; l < bot; ++l) down(l, std::true_type());
            bottom(std::true_type());
            for (int l = bot - 1; l >= lw; --l) up(l, std::true_type());
        }
        lds_sync<false>();
    } else {
        bottom(std::false_type());
    }
    for (int l = lw - 1; l >= 1; --l) up(l, std::false_type());

    A.template prolong<false>(T0, bot == 1 ? B : level(1), bot == 1, g.per, g.prolong);
    A.template smooth<false>(T0, g.nu2);
#pragma unroll
    for (int k = 0; k < kTopPairs; ++k)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int o = (c + A.y[k] + A.z[k]) & 1;
            if (A.on[k]) gu[top_elem(2 * A.m[k] + o, A.y[k], A.z[k])] = A.u[k][c];
        }
}

// Fills cc.g; returns the LDS bytes of k_coarse_fast, 0 where it does not
// apply (no room, or a level it cannot smooth).
template <class T>
int coarse_fast_layout(CoarseCycle<T>& cc) {
    CoarseGeom<T>& g = cc.g;
    g.nlev = cc.nlev;
    g.nu1 = cc.nu1;
    g.nu2 = cc.nu2;
    g.prolong = cc.prolong;
    g.pid = cc.pid;
    g.rtol = cc.rtol;
    g.iters = cc.iters;
    g.a = cc.L[0].box.a;
    const RBox& R = cc.L[0].box;
    g.H = R.H;
    g.GH = R.H * R.G[1];
    g.cs = (int)R.cstride;
    g.par = (R.lo[0] + R.lo[1] + R.lo[2]) & 1;
    g.u = cc.L[0].u + R.base;
    g.f = cc.L[0].f + R.base;
    size_t elems = 0;
    for (int l = 0; l < cc.nlev; ++l) {
        const RBox& B = cc.L[l].box;
        int cells = 1;
        bool even = true;
        for (int d = 0; d < 3; ++d) {
            g.n[l][d] = B.hi[d] - B.lo[d] + 1;
            g.c[l][d] = cc.L[l].fa.c[d];
            cells *= g.n[l][d];
            even = even && g.n[l][d] % 2 == 0 && (B.lo[d] & 1) == 0;
        }
        g.h[l] = cc.L[l].h;
        if (l + 1 < cc.nlev) {
            if (!even || !cc.L[l].push || cells > (l == 0 ? kMaxBottomCells : 2 * kCT)) return 0;
            elems += 2 * (size_t)cells + (l == 0 ? cells / 2 : 0);
        } else {
            if (l > 0 && cells > kCT) return 0;
            elems += cells;
        }
    }
    for (int d = 0; d < 3; ++d) g.per[d] = cc.per[d];
    const size_t N = (size_t)g.n[cc.nlev - 1][0] * g.n[cc.nlev - 1][1] * g.n[cc.nlev - 1][2];
    const size_t bytes = elems * sizeof(T) + 16 + 8 * N + 8 * 4 * (kCT / 64);
    return bytes + 2048 <= (size_t)lds_limit_bytes() ? (int)bytes : 0;
}
template int coarse_fast_layout<double>(CoarseCycle<double>&);
template int coarse_fast_layout<float>(CoarseCycle<float>&);

template <class T>
hipError_t launch_coarse_fast(hipStream_t s, const CoarseCycle<T>* cc, int n, const int* active, bool var,
                              int lds_bytes) {
    if (n <= 0) return hipSuccess;
    static const hipError_t once[2] = {
        hipFuncSetAttribute((const void*)k_coarse_fast<T, 0>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            lds_limit_bytes() - 2048),
        hipFuncSetAttribute((const void*)k_coarse_fast<T, 2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            lds_limit_bytes() - 2048)};
    (void)once;
    if (var) hipLaunchKernelGGL((k_coarse_fast<T, 2>), dim3(n), dim3(kCT), lds_bytes, s, cc, active);
    else hipLaunchKernelGGL((k_coarse_fast<T, 0>), dim3(n), dim3(kCT), lds_bytes, s, cc, active);
    return hipGetLastError();
}
template hipError_t launch_coarse_fast<double>(hipStream_t, const CoarseCycle<double>*, int, const int*, bool, int);
template hipError_t launch_coarse_fast<float>(hipStream_t, const CoarseCycle<float>*, int, const int*, bool, int);

}  // namespace bxmg
