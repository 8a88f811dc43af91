// Streaming pass of a Runge-Kutta stage for 3D meshes of affine elements
// (Sec. 2.2): per element the volume term and the flux bounce-back term of
// every moving velocity, the interior Runge-Kutta update and the element
// contributions of the boundary nodes.
//
// In an affine element dr_m/dx_k and J are constants, so the contravariant
// velocity c_m = sum_k e_k dr_m/dx_k is one number per velocity: neither the
// metric (9 values per node) nor 1/wJ is read. The pass works with L = -c .
// grad f itself; a contribution is scaled by wJ = w_i w_j w_k J where it is
// written. (Curved elements take k_stage23_mf, k_stage or k_stage_big: with the
// metric per node this split was slower there, 78 against 61 us on 1024
// elements of order 7. So do larger meshes of orders 2 to 4: affine_pass.)
//
// The unit of work is a pair of opposite velocities of one element (they share
// c up to its sign), with one thread per line of (N+1) nodes.
//
// Global memory is read and written in slot order (the interior block of a
// velocity is one run, face slots are runs of (N-1)^2 groups), each address
// computed once for all velocities: with the lines' own order instead the
// address units were the limit (20 cache accesses per instruction, 87% busy).
// A velocity's plane then passes through LDS (row stride N+1 or N+2, odd, so
// that a column of any direction meets every bank): every thread takes one
// line of each direction out of it, the r- and s-derivatives come back to the
// t-lines through two more planes, and the sum goes back to slot order. Per
// node and velocity that is 10 LDS accesses and 3 (N+1)/2 + O(1) multiply-adds
// (LineTab), against 26 and 3 (N+1) with one thread per node.
//
// Memory-bound: D3Q27 N = 7, 16^3 elements FP32 reads 280 MB and writes 263 MB by
// the counters (operand, f0, update, contributions) in 131 us, 4.1 TB/s, where a
// large copy reaches 4.9; L2 misses are 592 MB, and wavefronts wait 53% of their
// cycles. 12^3 FP64: 422 MB in 117 us. Per launch against the general kernels:
// D3Q27 N = 7 16^3 FP32 180 -> 131 us, 12^3 FP64 164 -> 117; D3Q19 N = 8 16^3 FP32 304 ->
// 161; N = 12 8^3 FP64 539 -> 121; N = 5 10^3 FP32 24 -> 19; N = 3 8^3 FP32 14 -> 8.
//
// A unit never waits for another one: with (N+1)^2 <= 64 lines it lives inside
// one wavefront and no workgroup barrier is left, so the loads of some units
// run under the arithmetic of others.
#pragma once

#include "kernels_impl.h"

namespace sel {

// A centro-(anti)symmetric (N+1) x (N+1) line operator M (M[N-i][N-q] = -+
// M[i][q]) by sums and differences of mirrored values, s_q = x_q + x_{N-q}, d_q =
// x_q - x_{N-q} (q < h = (N+1)/2):
//   E_i = sum A_iq s_q, O_i = sum B_iq d_q, A_iq = (M_iq + M_i,N-q)/2, B_iq = (M_iq - M_i,N-q)/2,
//   (M x)_i = E_i + O_i and (M x)_{N-i} = -+(E_i - O_i).
// The rows of M sum to zero, so the sums are taken relative to the innermost
// pair (the middle node when N + 1 is odd): constant lines give exactly zero
// whatever the rounding of the table, and rounding acts at the size of the
// variation along the line, not at the level of the populations.
// A and B lie in constant memory and are read as wavefront-uniform scalars.
template <int n1>
struct LineTab {
    static constexpr int h = n1 / 2, odd = n1 % 2, na = odd ? h : h - 1;
    static constexpr int rows = h + odd;          // row h: the middle node
    static constexpr int nA = rows * na, nB = rows * h, size = nA + nB;
};

// M[n1 x n1] with rows summing to zero (the derivative matrix, or filter - identity)
template <int n1>
void line_tab(const double *M, double *t)
{
    using L = LineTab<n1>;
    for (int i = 0; i < L::rows; ++i)
        for (int q = 0; q < L::h; ++q) {
            const double a = M[i * n1 + q], b = M[i * n1 + n1 - 1 - q];
            if (q < L::na) t[i * L::na + q] = 0.5 * (a + b);
            t[L::nA + i * L::h + q] = 0.5 * (a - b);
        }
}

// place of shared group g in the state: tiles of 64 groups (SIdx)
template <int Q>
__device__ __forceinline__ int64_t tile_at(uint32_t g)
{
    return (int64_t)(g / kTile) * (Q * kTile) + (g % kTile);
}

template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T *;

// y = D x for the antisymmetric derivative matrix
template <int n1, typename T>
__device__ __forceinline__ void line_derivative(const T (&x)[n1], T (&y)[n1], ConstPtr<T> t)
{
    using L = LineTab<n1>;
    constexpr int h = L::h, na = L::na;
    // tables that don't fit the scalar registers beside the rest are read in
    // place instead of being held (and spilled) over the loop
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
    for (int i = 0; i < h; ++i) {
        T E = T(0), O = t[L::nA + i * h] * d[0];
        if constexpr (na > 0) E = t[i * na] * s[0];
#pragma unroll
        for (int q = 1; q < na; ++q) E += t[i * na + q] * s[q];
#pragma unroll
        for (int q = 1; q < h; ++q) O += t[L::nA + i * h + q] * d[q];
        y[i] = O + E;
        y[n1 - 1 - i] = O - E;
    }
    if constexpr (L::odd) {
        T O = t[L::nA + h * h] * d[0];
#pragma unroll
        for (int q = 1; q < h; ++q) O += t[L::nA + h * h + q] * d[q];
        y[h] = O;
    }
}

template <int N, int Q, typename T>
struct StreamGeo {
    static constexpr int n1 = N + 1, NL = n1 * n1, NP = NL * n1;
    static constexpr int NI = (N - 1) * (N - 1) * (N - 1), NB = NP - NI;
    static constexpr int RS = n1 | 1, PL = RS * NL;  // row stride and plane in LDS
    static constexpr int NPAIR = (Q - 1) / 2;
    // whole units inside a wavefront when their lines fill at least three
    // quarters of it; else units side by side in a workgroup of up to 256
    // threads (512 above 128 lines), as many as leave the fewest idle threads
    // over the passes that all pairs take, within 56 KB of LDS
    static constexpr int UPW = 64 / NL;
    static constexpr bool WAVE = UPW * NL >= 48;
    static constexpr int units_for(int u) { return ((u * NL + 63) / 64) * 64; }
    static constexpr int best_units()
    {
        int best = 1;
        double eff = 0.0;
        for (int u = 1; u <= NPAIR; ++u) {
            const int b = units_for(u);
            if (u > 1 && (b > (NL > 128 ? 512 : 256) || 3 * u * PL * (int)sizeof(T) > 56 * 1024)) break;
            const int passes = (NPAIR + u - 1) / u;
            const double f = double(NPAIR * NL) / double(passes * b);
            if (f > eff) {
                eff = f;
                best = u;
            }
        }
        return best;
    }
    // 4 wavefronts, or in FP32 5 where that is one pass instead of a nearly
    // empty second (N = 4, D3Q19, 20^3 elements 1075 -> 1062 us in three steps;
    // FP64 16^3 914 -> 975: not there)
    static constexpr int wave_count() { return (NPAIR + UPW - 1) / UPW <= (sizeof(T) == 4 ? 5 : 4) ? (NPAIR + UPW - 1) / UPW : 4; }
    static constexpr int UPB_()
    {
        if constexpr (WAVE) return wave_count() * UPW;
        else return best_units();
    }
    static constexpr int UPB = UPB_();
    static constexpr int BLOCK = WAVE ? (UPB / (UPW > 0 ? UPW : 1)) * 64 : units_for(UPB);
    static constexpr int PASSES = (NPAIR + UPB - 1) / UPB;
    // slots of a thread: interior slots as vectors of VW values where the
    // interior block of every velocity starts on a multiple of 16 bytes
    static constexpr int VW = (NI * sizeof(T)) % 16 == 0 ? 16 / sizeof(T) : 1;
    static constexpr int NIR = (NI / VW + NL - 1) / NL, NBR = (NB + NL - 1) / NL;
};

template <int N, int Q, typename T>
struct StreamArgs {
    static constexpr int NPAIR = (Q - 1) / 2;
    const T *op;    // operand state fk
    const T *f0in;  // post-collision state
    T *out;         // out = ca f0 + cb fk + cc L(fk), interior nodes
    T *rtb;         // element contributions of boundary nodes [Q][plane]
    const T *rhoc, *wallu;
    const T *aff;   // [E][10] dr_m/dx_k, J
    const T *tab;   // LineTab of the derivative matrix
    const T *Fn;    // force density per node id [Gtot][3] (nullptr: none)
    const int32_t *bpos, *bmap, *posmap, *ftag;
    int64_t E, QGi, plane;
    T ca, cb, cc, rho0;
    int incr;       // ca + cb = 1: increment form (rk_combine)
    int body;       // some pf is not zero
    int same;       // f0in is op: read once
    int split;      // workgroups an element's pairs are dealt to
    T w[N + 1];     // GLL weights
    int32_t pa[NPAIR], pb[NPAIR];  // velocities of each pair, e_pb = -e_pa
    T pe[NPAIR][3], pt[NPAIR], pf[NPAIR];  // e, weight and F* per unit density of pa
};

// WALL: some face of the mesh is a wall (compiled apart: the wall flux takes 35
// registers, which the meshes without walls turn into a fifth wave per SIMD).
template <int N, int Q, typename T, bool WALL>
__global__ void __launch_bounds__((StreamGeo<N, Q, T>::BLOCK), (sizeof(T) == 4 && N <= 8 ? (WALL ? 3 : 4) : 2))
    k_stream(StreamArgs<N, Q, T> A)
{
    using SG = StreamGeo<N, Q, T>;
    constexpr int n1 = SG::n1, NL = SG::NL, NP = SG::NP, NI = SG::NI, NB = SG::NB, RS = SG::RS, PL = SG::PL;
    constexpr int NPAIR = SG::NPAIR, M1 = N - 1;
    __shared__ T lds[SG::UPB][3][PL];

    const uint32_t tid = threadIdx.x;
    const int64_t wg = xcd_block(A.E * A.split);
    if (wg >= A.E * A.split) return;  // whole workgroup
    const int64_t e = A.split == 1 ? wg : wg / A.split;
    const uint32_t part = (uint32_t)(wg - e * A.split);
    uint32_t unit, line;
    bool act;
    if constexpr (SG::WAVE) {
        const uint32_t w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
        unit = (SG::UPW == 1) ? w : w * SG::UPW + l / NL;
        line = (SG::UPW == 1) ? l : l % NL;
        act = l < SG::UPW * NL;
    } else {
        unit = tid / NL;
        line = tid - unit * NL;
        act = tid < SG::UPB * NL;
    }
    if (!act) {
        unit = 0;
        line = 0;
    }
    auto sync = [] {
        if constexpr (SG::WAVE) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };
    const int64_t ib = e * (int64_t)Q * NI;
    const ConstPtr<T> tab = (ConstPtr<T>)A.tab;
    const ConstPtr<T> ga = (ConstPtr<T>)(A.aff + e * 10);

    // the rest velocity neither streams nor meets a wall
    for (uint32_t s = part ? NI : tid; s < NI; s += SG::BLOCK) {
        const T v = A.op[ib + s];
        A.out[ib + s] = rk_combine(A.ca, A.cb, A.cc, A.f0in[ib + s], v, T(0), A.incr);
    }

    // the thread's slots: position in the LDS planes, and for boundary slots
    // the group's place in the state, the place of the contribution and the
    // faces through the node
    constexpr int VW = SG::VW, NIR = SG::NIR, NBR = SG::NBR;
    typedef T vec __attribute__((ext_vector_type(VW > 1 ? VW : 2)));
    uint32_t ip[NIR * VW], bp[NBR], grp[NBR], slot[NBR];
    uint32_t wcode[NBR];  // 8 bits per direction: wall tag, bit 7 for the face r_m = +1
    T wb[NBR];  // wJ
#pragma unroll
    for (int r = 0; r < NIR * VW; ++r) {
        const uint32_t s = min(VW * (line + NL * (r / VW)) + r % VW, (uint32_t)NI - 1);
        ip[r] = (s % M1 + 1) + RS * (s / M1 % M1 + 1) + RS * n1 * (s / (M1 * M1) + 1);
    }
    const int32_t *ft = A.ftag + e * 6;
    const bool wall = WALL && (ft[0] | ft[1] | ft[2] | ft[3] | ft[4] | ft[5]);
#pragma unroll
    for (int r = 0; r < NBR; ++r) {
        const uint32_t b = min(line + NL * r, (uint32_t)NB - 1);
        grp[r] = A.bmap[e * NB + b];
        slot[r] = A.posmap[e * NB + b];
        const uint32_t p = A.bpos[b], x[3] = {p % n1, p / n1 % n1, p / NL};
        bp[r] = x[0] + RS * (x[1] + n1 * x[2]);
        wb[r] = A.w[x[0]] * A.w[x[1]] * A.w[x[2]] * ga[9];
        wcode[r] = 0;
        if (wall) {
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const uint32_t tag = (x[m] == 0) ? ft[2 * m] : (x[m] == N) ? ft[2 * m + 1] : 0;
                if (tag) wcode[r] |= (tag | (x[m] == N ? 0x80u : 0u)) << (8 * m);
            }
        }
    }
    const uint32_t i = line % n1, j = line / n1;
    T *P = &lds[unit][0][0], *R1 = &lds[unit][1][0], *R2 = &lds[unit][2][0];
    const uint32_t pt0 = i + RS * j, pr0 = RS * line, ps0 = i + RS * n1 * j;


    // a velocity's values in the thread's slots: operand and, for the interior,
    // the post-collision state
    struct Vals {
        T vi[NIR * VW], f0[NIR * VW], vb[NBR];
    };
    uint32_t ln = line;
    auto load = [&](Vals &V, uint32_t a) {
        // addresses are formed where they are used (hoisted out of the loop over
        // the pairs they would hold most registers)
#pragma unroll
        for (int r = 0; r < NBR; ++r) asm volatile("" : "+v"(grp[r]), "+v"(slot[r]));

        asm volatile("" : "+v"(ln));
        const T *q = A.op + (ib + a * (uint32_t)NI), *z = A.f0in + (ib + a * (uint32_t)NI);
        const T *qb = A.op + (A.QGi + a * (uint32_t)kTile);
        auto interior = [&](const T *p, T (&v)[NIR * VW]) {
#pragma unroll
            for (int r = 0; r < NIR; ++r) {
                const uint32_t s = min(ln + NL * r, (uint32_t)(NI / VW) - 1);
                if constexpr (VW > 1) {
                    const vec x = __builtin_nontemporal_load(reinterpret_cast<const vec *>(p) + s);
#pragma unroll
                    for (int c = 0; c < VW; ++c) v[r * VW + c] = x[c];
                } else {
                    v[r] = __builtin_nontemporal_load(p + s);
                }
            }
        };
        interior(q, V.vi);
        if (!A.same) interior(z, V.f0);
#pragma unroll
        for (int r = 0; r < NBR; ++r) V.vb[r] = qb[tile_at<Q>(grp[r])];
    };

    // velocity a of pair pi with the values V; u = 1 for the pair's second one
    auto velocity = [&](auto U, uint32_t pi, bool on, const Vals &V) {
        constexpr int u = decltype(U)::value;
        const T sg = u ? T(1) : T(-1);  // rt = -c . grad f, c of the pair's second velocity is -c
        const T ex = A.pe[pi][0], ey = A.pe[pi][1], ez = A.pe[pi][2];
        const uint32_t a = u ? A.pb[pi] : A.pa[pi];
        // c_m of the pair's first velocity
        T c[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) c[m] = ex * ga[3 * m] + ey * ga[3 * m + 1] + ez * ga[3 * m + 2];
        if (on) {
#pragma unroll
            for (int r = 0; r < NIR * VW; ++r)
                if (NI % (NL * VW) == 0 || r / VW + 1 < NIR || ln + NL * (r / VW) < NI / VW) P[ip[r]] = V.vi[r];
#pragma unroll
            for (int r = 0; r < NBR; ++r)
                if (r + 1 < NBR || ln + NL * r < NB) P[bp[r]] = V.vb[r];
        }
        sync();
        T rt[n1];
        {
            T x[n1], y[n1];
#pragma unroll
            for (int q = 0; q < n1; ++q) x[q] = P[pr0 + q];
            line_derivative<n1, T>(x, y, tab);
            if (act) {
#pragma unroll
                for (int q = 0; q < n1; ++q) R1[pr0 + q] = y[q];
            }
#pragma unroll
            for (int q = 0; q < n1; ++q) x[q] = P[ps0 + RS * q];
            line_derivative<n1, T>(x, y, tab);
            if (act) {
#pragma unroll
                for (int q = 0; q < n1; ++q) R2[ps0 + RS * q] = y[q];
            }
#pragma unroll
            for (int q = 0; q < n1; ++q) x[q] = P[pt0 + RS * n1 * q];
            line_derivative<n1, T>(x, rt, tab);
        }
        sync();
#pragma unroll
        for (int k = 0; k < n1; ++k) {
            const uint32_t x = pt0 + RS * n1 * k;
            rt[k] = sg * (c[0] * R1[x] + c[1] * R2[x] + c[2] * rt[k]);
        }
        if (act) {
#pragma unroll
            for (int k = 0; k < n1; ++k) R1[pt0 + RS * n1 * k] = rt[k];
        }
        sync();
        if (!on) return;
        // interior: out = ca f0 + cb fk + cc (L + F*)
        T *o = A.out + (ib + a * (uint32_t)NI);
        const T pf = -sg * A.pf[pi], t3 = -sg * T(3) * A.pt[pi];
#pragma unroll
        for (int r = 0; r < NIR; ++r) {
            const uint32_t s = ln + NL * r;
            if (!(NI % (NL * VW) == 0 || r + 1 < NIR || s < NI / VW)) continue;
            vec y;
#pragma unroll
            for (int v = 0; v < VW; ++v) {
                const int64_t id = e * NI + (s * VW + v);
                T L = R1[ip[r * VW + v]];
                if (A.body) L += pf * A.rhoc[id];
                if (A.Fn) L += t3 * (ex * A.Fn[3 * id] + ey * A.Fn[3 * id + 1] + ez * A.Fn[3 * id + 2]);
                y[v] = rk_combine(A.ca, A.cb, A.cc, A.same ? V.vi[r * VW + v] : V.f0[r * VW + v], V.vi[r * VW + v], L,
                                  A.incr);
            }
            if constexpr (VW > 1) __builtin_nontemporal_store(y, reinterpret_cast<vec *>(o) + s);
            else o[s] = y[0];
        }
        // boundary: the element's contribution, wJ L
        T b[NBR];
#pragma unroll
        for (int r = 0; r < NBR; ++r) b[r] = R1[bp[r]];
        if (wall) {
            // flux bounce-back on the wall faces through the node where the
            // velocity enters the element (n . e < 0), with the outward area
            // vector +-(w_end)^-1 wJ dr_m/dx of the face r_m = +-1: the
            // population meets the reflected one, f_a - f_b - 2 t_a rho0 (e_a .
            // u_w)/c_s^2
            const uint32_t ao = u ? A.pa[pi] : A.pb[pi];
#pragma unroll
            for (int r = 0; r < NBR; ++r) {
                if (!wcode[r]) continue;
                const T vr = A.op[A.QGi + ao * (uint32_t)kTile + tile_at<Q>(grp[r])];
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    const uint32_t code = (wcode[r] >> (8 * m)) & 0xffu;
                    if (code == 0) continue;
                    const T ne = ((code & 0x80u) ? -sg : sg) * T(N * (N + 1)) / T(2) * c[m];
                    if (!(ne < T(0))) continue;
                    const T *ub = A.wallu + 3 * (code & 0x7fu);
                    const T vo = vr - sg * T(6) * A.pt[pi] * A.rho0 * (ex * ub[0] + ey * ub[1] + ez * ub[2]);
                    b[r] += ne * (V.vb[r] - vo);
                }
            }
        }
        T *rb = A.rtb + (int64_t)a * A.plane;
#pragma unroll
        for (int r = 0; r < NBR; ++r)
            if (r + 1 < NBR || ln + NL * r < NB) rb[slot[r]] = b[r] * wb[r];
    };

    // the next velocity's values are loaded while one is streamed
    auto pair_of = [&](uint32_t it, bool &on) {
        const uint32_t pr = (it * A.split + part) * SG::UPB + unit;
        on = act && pr < NPAIR;
        return on ? pr : 0u;
    };
    Vals va, vb;
    bool on;
    uint32_t pi = pair_of(0, on);
    if (on) load(va, A.pa[pi]);
    for (uint32_t it = 0; (it * A.split + part) * SG::UPB < NPAIR; ++it) {
        if constexpr (SG::WAVE) {
            if (__builtin_amdgcn_readfirstlane((it * A.split + part) * SG::UPB + unit) >= NPAIR) break;
        }
        if (on) load(vb, A.pb[pi]);
        velocity(std::integral_constant<int, 0>{}, pi, on, va);
        bool on2;
        const uint32_t p2 = pair_of(it + 1, on2);
        if (on2) load(va, A.pa[p2]);
        velocity(std::integral_constant<int, 1>{}, pi, on, vb);
        pi = p2;
        on = on2;
    }
}

}  // namespace sel
