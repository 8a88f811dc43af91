// Modal filter and collision of 3D meshes (Secs. 2.2.3 and 2.1), ahead of the
// streaming of the first Runge-Kutta stage. (Curved meshes for which
// Impl::first_stage holds take the filter alone from here, or neither.)
//
// k_relax: one workgroup holds all Q planes of an element (several small
// elements) in LDS. A thread loads its slots for every velocity, the filter
// runs along lines in place (one thread per line, LineTab of F - 1; the plane's
// row stride is odd, so lines of every direction are free of bank conflicts),
// and the thread collides its slots and stores them: the state is read and
// written once. Filter rows take n1 LDS reads and n1 writes per line instead of
// n1 reads per node. Used where two workgroups fit the 160 KB of a CU.
// k_filter + k_collide: the same in two passes over the state where the planes
// don't fit (FP64 from N = 7, N = 12): lines of one velocity per unit, then one
// thread per node id. k_collide alone serves a step without a pending filter.
// Measured on affine meshes against filter, collision and streaming in one
// kernel (up to 76 KB of LDS and 500 B of spills), as relaxation + streaming
// pass: D3Q27 N = 7, 16^3 FP32 307 -> 98 + 125 us (3.9 TB/s); 12^3 FP64
// 276 -> 62 + 42 + 100 (5.1 and 6 TB/s; k_relax with one workgroup per CU 103);
// D3Q19 N = 8, 16^3 FP32 474 -> 102 + 145 (in two passes 151 + 57); N = 12, 8^3
// FP64 889 -> 95 + 47 + 110. The filter at the end of a call: 152 -> 81, 142 -> 62,
// 161 -> 97 and 250 -> 95 us.
// The filter is taken as the identity plus a small correction: only the
// correction is rounded, at the size of the variation along the line.
#pragma once

#include "kernels_stream.h"

namespace sel {

// x += (F - 1) x along a line; the end nodes keep their values
template <int n1, typename T>
__device__ __forceinline__ void line_filter(T (&x)[n1], ConstPtr<T> t)
{
    using L = LineTab<n1>;
    constexpr int h = L::h, na = L::na;
    if constexpr (L::size * sizeof(T) > 160) asm volatile("" : "+s"(t));
    T s[h], d[h];
#pragma unroll
    for (int q = 0; q < h; ++q) {
        s[q] = x[q] + x[n1 - 1 - q];
        d[q] = x[q] - x[n1 - 1 - q];
    }
    const T ref = L::odd ? x[h] + x[h] : s[h - 1];
#pragma unroll
    for (int q = 0; q < na; ++q) s[q] -= ref;
#pragma unroll
    for (int i = 1; i < L::rows; ++i) {
        T E = T(0);
        if constexpr (na > 0) E = t[i * na] * s[0];
#pragma unroll
        for (int q = 1; q < na; ++q) E += t[i * na + q] * s[q];
        if (i == h) {
            x[h] += E;
            continue;
        }
        T O = t[L::nA + i * h] * d[0];
#pragma unroll
        for (int q = 1; q < h; ++q) O += t[L::nA + i * h + q] * d[q];
        x[i] += E + O;
        x[n1 - 1 - i] += E - O;
    }
}

template <typename T>
struct RelaxArgs {
    const T *op;     // state
    T *out;          // post-collision state, or the filtered state
    T *rhoc;         // density at the collision [Gtot]
    const T *tab;    // LineTab of the filter minus the identity
    const T *Fn;     // force density per node id [Gtot][3] (nullptr: none)
    const float *dtau;  // closure increments per node id (nullptr: none)
    const int32_t *bpos, *bmap;
    const uint8_t *bown;
    int64_t E, Gi, Gtot, QGi;
    T dt, omega, tau, rho0, g[3];
    int split;  // k_filter: workgroups an element's velocities are dealt to
};

// collision of one node with its body force, force per node and closure increment
template <int Q, typename T, bool DEV>
__device__ __forceinline__ void relax_node(const RelaxArgs<T> &A, T (&v)[Q], int64_t id, T &rho)
{
    const T om = A.dtau ? T(1) / (A.tau + T(A.dtau[id]) + T(0.5)) : A.omega;
    T F[3] = {};
    if (A.Fn) {
#pragma unroll
        for (int c = 0; c < 3; ++c) F[c] = A.Fn[3 * id + c];
    }
    collide_node<3, Q, T, DEV>(v, A.rho0, om, A.dt, A.g, rho, F, A.Fn != nullptr);
}

template <int N, int Q, typename T>
struct RelaxGeo {
    using SG = StreamGeo<N, Q, T>;
    static constexpr int n1 = SG::n1, NL = SG::NL, NP = SG::NP, NI = SG::NI, NB = SG::NB, RS = SG::RS, PL = SG::PL;
    static constexpr int PLANES = Q * PL * (int)sizeof(T);
    static constexpr bool FUSED = PLANES <= 80 * 1024;
    // elements per workgroup: about 256 slots, within 40 KB
    static constexpr int EPB = (NP >= 128 || !FUSED) ? 1 : (256 / NP * PLANES <= 40 * 1024 ? 256 / NP : 40 * 1024 / PLANES);
    static constexpr int SLOTS = EPB * NP;
    // 4 or 8 wavefronts, a multiple of the SIMDs (with 6, a second workgroup
    // found no place on the SIMDs that hold 2 of the first: N = 8 ran at 1.4
    // wavefronts per SIMD)
    static constexpr int BLOCK = SLOTS <= 256 ? 256 : 512;
    static constexpr int R = (SLOTS + BLOCK - 1) / BLOCK;  // slots per thread
};

template <int N, int Q, typename T, bool DEV, bool COLLIDE>
__global__ void __launch_bounds__((RelaxGeo<N, Q, T>::BLOCK), (sizeof(T) == 4 ? 4 : 1)) k_relax(RelaxArgs<T> A)
{
    using G = RelaxGeo<N, Q, T>;
    constexpr int n1 = G::n1, NL = G::NL, NP = G::NP, NI = G::NI, NB = G::NB, RS = G::RS, PL = G::PL, R = G::R,
                  EPB = G::EPB, BLOCK = G::BLOCK, M1 = N - 1;
    __shared__ T lds[EPB * Q * PL];
    const uint32_t tid = threadIdx.x;
    const int64_t nblk = (A.E + EPB - 1) / EPB, eb = xcd_block(nblk);
    if (eb >= nblk) return;  // whole workgroup
    const ConstPtr<T> tab = (ConstPtr<T>)A.tab;

    bool ok[R], own[R];
    uint32_t pos[R], st[R];
    int64_t base[R], id[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t q = tid + r * BLOCK, le = q / NP, s = q % NP;
        const int64_t e = eb * EPB + le;
        ok[r] = q < G::SLOTS && e < A.E;
        own[r] = ok[r];
        pos[r] = st[r] = 0;
        base[r] = id[r] = 0;
        if (!ok[r]) continue;
        if (s < NI) {
            pos[r] = (s % M1 + 1) + RS * (s / M1 % M1 + 1) + RS * n1 * (s / (M1 * M1) + 1);
            base[r] = e * (int64_t)(Q * NI) + s;
            id[r] = e * NI + s;
            st[r] = NI;
        } else {
            const uint32_t b = s - NI, p = A.bpos[b], g = A.bmap[e * NB + b];
            pos[r] = p % n1 + RS * (p / n1);
            base[r] = A.QGi + tile_at<Q>(g);
            id[r] = A.Gi + g;
            st[r] = kTile;
            own[r] = A.bown[e * NB + b] != 0;
        }
        pos[r] += le * (Q * PL);
        T v[Q];
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            v[a] = A.op[base[r] + a * st[r]];
        });
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            lds[pos[r] + a * PL] = v[a];
        });
    }
    __syncthreads();
    static_for<0, 3>([&](auto MM) {
        constexpr int m = decltype(MM)::value;
        constexpr int LINES = EPB * Q * NL, str = (m == 0) ? 1 : (m == 1) ? RS : RS * n1;
        for (uint32_t x = tid; x < LINES; x += BLOCK) {
            const uint32_t l = x % NL;
            T *P = lds + x / NL * PL + ((m == 0) ? RS * l : l % n1 + l / n1 * ((m == 1) ? RS * n1 : RS));
            T y[n1];
#pragma unroll
            for (int q = 0; q < n1; ++q) y[q] = P[str * q];
            line_filter<n1, T>(y, tab);
#pragma unroll
            for (int q = 1; q < N; ++q) P[str * q] = y[q];
        }
        __syncthreads();
    });
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!own[r]) continue;
        T v[Q];
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            v[a] = lds[pos[r] + a * PL];
        });
        if constexpr (COLLIDE) {
            T rho;
            relax_node<Q, T, DEV>(A, v, id[r], rho);
            A.rhoc[id[r]] = rho;
        }
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            A.out[base[r] + a * st[r]] = v[a];
        });
    }
}

// The filter alone, velocity by velocity: a unit is one velocity of one
// element with a thread per line (units as in k_stream, one plane each).
template <int N, int Q, typename T>
struct FilterGeo {
    using SG = StreamGeo<N, Q, T>;
    static constexpr int NL = SG::NL, UPW = SG::UPW;
    static constexpr bool WAVE = SG::WAVE;
    static constexpr int UPB = WAVE ? 4 * UPW : (NL > 128 ? 3 : 256 / NL);
    static constexpr int BLOCK = WAVE ? 256 : (UPB * NL + 63) / 64 * 64;
};

template <int N, int Q, typename T>
__global__ void __launch_bounds__((FilterGeo<N, Q, T>::BLOCK)) k_filter(RelaxArgs<T> A)
{
    using SG = StreamGeo<N, Q, T>;
    using G = FilterGeo<N, Q, T>;
    constexpr int n1 = SG::n1, NL = SG::NL, NI = SG::NI, NB = SG::NB, RS = SG::RS, PL = SG::PL, M1 = N - 1;
    constexpr int NIR = (NI + NL - 1) / NL, NBR = SG::NBR;
    __shared__ T lds[G::UPB][PL];
    const uint32_t tid = threadIdx.x;
    const int64_t wg = xcd_block(A.E * A.split);
    if (wg >= A.E * A.split) return;  // whole workgroup
    const int64_t e = A.split == 1 ? wg : wg / A.split;
    const uint32_t part = (uint32_t)(wg - e * A.split);
    uint32_t unit, line;
    bool act;
    if constexpr (G::WAVE) {
        const uint32_t w = tid >> 6, l = tid & 63;
        unit = w * G::UPW + l / NL;
        line = l % NL;
        act = l < G::UPW * NL;
    } else {
        unit = tid / NL;
        line = tid - unit * NL;
        act = tid < G::UPB * NL;
    }
    if (!act) unit = line = 0;
    auto sync = [] {
        if constexpr (G::WAVE) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };
    const ConstPtr<T> tab = (ConstPtr<T>)A.tab;
    uint32_t ip[NIR], bp[NBR], grp[NBR];
    bool own[NBR];
#pragma unroll
    for (int r = 0; r < NIR; ++r) {
        const uint32_t s = min(line + NL * r, (uint32_t)NI - 1);
        ip[r] = (s % M1 + 1) + RS * (s / M1 % M1 + 1) + RS * n1 * (s / (M1 * M1) + 1);
    }
#pragma unroll
    for (int r = 0; r < NBR; ++r) {
        const uint32_t b = min(line + NL * r, (uint32_t)NB - 1), p = A.bpos[b];
        grp[r] = A.bmap[e * NB + b];
        own[r] = line + NL * r < NB && A.bown[e * NB + b];
        bp[r] = p % n1 + RS * (p / n1);
    }
    T *P = lds[unit];
    const uint32_t i = line % n1, j = line / n1;
    for (uint32_t a0 = part * G::UPB; a0 < Q; a0 += A.split * G::UPB) {
        const uint32_t a = a0 + unit;
        const bool on = act && a < Q;
        const T *q = A.op + e * (int64_t)(Q * NI) + (on ? a : 0) * (uint32_t)NI;
        const T *qb = A.op + A.QGi + (on ? a : 0) * (uint32_t)kTile;
        T vi[NIR], vb[NBR];
#pragma unroll
        for (int r = 0; r < NIR; ++r) vi[r] = q[min(line + NL * r, (uint32_t)NI - 1)];
#pragma unroll
        for (int r = 0; r < NBR; ++r) vb[r] = qb[tile_at<Q>(grp[r])];
        if (on) {
#pragma unroll
            for (int r = 0; r < NIR; ++r)
                if (line + NL * r < NI) P[ip[r]] = vi[r];
#pragma unroll
            for (int r = 0; r < NBR; ++r)
                if (line + NL * r < NB) P[bp[r]] = vb[r];
        }
        sync();
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const uint32_t o = (m == 0) ? RS * line : i + j * ((m == 1) ? RS * n1 : RS);
            const int str = (m == 0) ? 1 : (m == 1) ? RS : RS * n1;
            T y[n1];
#pragma unroll
            for (int k = 0; k < n1; ++k) y[k] = P[o + str * k];
            line_filter<n1, T>(y, tab);
            if (on) {
#pragma unroll
                for (int k = 1; k < N; ++k) P[o + str * k] = y[k];
            }
            sync();
        }
        if (on) {
            T *o = A.out + e * (int64_t)(Q * NI) + a * (uint32_t)NI, *ob = A.out + A.QGi + a * (uint32_t)kTile;
#pragma unroll
            for (int r = 0; r < NIR; ++r)
                if (line + NL * r < NI) o[line + NL * r] = P[ip[r]];
#pragma unroll
            for (int r = 0; r < NBR; ++r)
                if (own[r]) ob[tile_at<Q>(grp[r])] = P[bp[r]];
        }
        sync();  // the plane is read before the next velocity fills it
    }
}

// Moments of 3D meshes at every element node, FP64 (Eqs. pressure, momentum).
// The populations are read in slot order, as runs, and the results go through
// LDS to be written as runs in node order (one thread per node in node order
// read six slots to a run and wrote 24-byte pieces: 16^3 elements N = 7 FP32 78
// us, here 59; D3Q19 N = 8 89 and 69; 12^3 N = 7 FP64 41 and 33.5). Elements of more
// than 1024 nodes take 1024 threads (N = 12 6^3 FP64: 17.9 us with 256, here 14.1).
template <int N>
struct MomentGeo {
    static constexpr int NP = (N + 1) * (N + 1) * (N + 1), EPB = NP >= 256 ? 1 : 256 / NP;
    static constexpr int BLOCK = NP > 1024 ? 1024 : 256;
};
template <int N, int Q, typename T, bool DEV>
__global__ void __launch_bounds__(MomentGeo<N>::BLOCK) k_moments_el(const T *f, const int32_t *bpos, const int32_t *bmap, int64_t E,
                                                    int64_t QGi, double rho0, double *rho, double *u)
{
    using SG = StreamGeo<N, Q, T>;
    constexpr int n1 = SG::n1, NP = SG::NP, NI = SG::NI, NB = SG::NB, M1 = N - 1, EPB = MomentGeo<N>::EPB,
                  BLOCK = MomentGeo<N>::BLOCK;
    __shared__ double sm[4][EPB * NP];
    const int64_t nblk = (E + EPB - 1) / EPB, eb = xcd_block(nblk);
    if (eb >= nblk) return;  // whole workgroup
    const int64_t left = E - eb * EPB;
    const uint32_t nodes = (left < EPB ? (int)left : EPB) * NP;
    for (uint32_t q = threadIdx.x; q < nodes; q += BLOCK) {
        const uint32_t le = q / NP, s = q % NP;
        const int64_t e = eb * EPB + le;
        uint32_t p, st;
        int64_t base;
        if (s < NI) {
            p = (s % M1 + 1) + n1 * (s / M1 % M1 + 1) + n1 * n1 * (s / (M1 * M1) + 1);
            base = e * (int64_t)(Q * NI) + s;
            st = NI;
        } else {
            p = bpos[s - NI];
            base = QGi + tile_at<Q>(bmap[e * NB + s - NI]);
            st = kTile;
        }
        double m = 0, j[3] = {0, 0, 0};
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            const double v = double(f[base + a * st]);
            m += v;
            if constexpr (lat_e<3, Q>(a, 0) != 0) j[0] += lat_e<3, Q>(a, 0) * v;
            if constexpr (lat_e<3, Q>(a, 1) != 0) j[1] += lat_e<3, Q>(a, 1) * v;
            if constexpr (lat_e<3, Q>(a, 2) != 0) j[2] += lat_e<3, Q>(a, 2) * v;
        });
        const double r = DEV ? rho0 + m : m;
        p += le * NP;
        sm[0][p] = r;
        double *su = &sm[1][0] + 3 * p;
        for (int c = 0; c < 3; ++c) su[c] = j[c] / r;
    }
    __syncthreads();
    const int64_t o = eb * EPB * NP;
    for (uint32_t q = threadIdx.x; q < nodes; q += BLOCK) rho[o + q] = sm[0][q];
    for (uint32_t q = threadIdx.x; q < 3 * nodes; q += BLOCK) u[3 * o + q] = (&sm[1][0])[q];
}

// The collision alone, one thread per node id. op and out may be the same.
template <int N, int Q, typename T, bool DEV>
__global__ void __launch_bounds__(256) k_collide(RelaxArgs<T> A)
{
    constexpr int NI = (N - 1) * (N - 1) * (N - 1);
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= A.Gtot) return;
    const SIdx si = sidx_node(id, A.Gi, NI, Q, A.QGi);
    T v[Q], rho;
    static_for<0, Q>([&](auto AA) {
        constexpr int a = decltype(AA)::value;
        v[a] = A.op[si.base + (int64_t)a * si.stride];
    });
    relax_node<Q, T, DEV>(A, v, id, rho);
    A.rhoc[id] = rho;
    static_for<0, Q>([&](auto AA) {
        constexpr int a = decltype(AA)::value;
        A.out[si.base + (int64_t)a * si.stride] = v[a];
    });
}

}  // namespace sel
