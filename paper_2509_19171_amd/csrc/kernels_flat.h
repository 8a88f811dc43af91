// Stage kernels of small 2D meshes (D2Q9; sel::flat_2d says which). A launch of
// a few microseconds costs as much as its work there, so a stage is one kernel:
// the shared-node assembly of a stage is done by the kernel of the next one,
// which reads the contributions of a boundary node's members and combines them
// itself (every copy the same way; the owning copy stores the value where a
// later stage needs it). A separate assembly doubles the launches: 64 elements
// N = 5 FP64 took 6.3 + 4.0 us per stage, 1024 elements N = 7 FP32 7.4 + 4.8.
//
// What a kernel reads of other elements' boundary nodes (the contributions of
// the last stage and the two states it combines) no kernel writes at the same
// time: contributions and densities alternate between two buffers, and the new
// post-collision state takes the array whose boundary part is not in use (the
// callers in launch_impl.h keep the roles).
//
// One thread per node and all velocities in registers; the node table [E][NP]
// (interior slot or group, contribution slot, members and owner, extra rank
// index) makes every address known after one load. Blocks of about one
// wavefront: the smallest meshes still spread over the chip. With the
// discontinuous coupling a node has one copy and nothing is pending: the assembly
// with the interface flux stays a kernel of its own.
#pragma once

#include "kernels_impl.h"

namespace sel {

// node table entry: x interior slot or group, y contribution slot, z members of
// the group (0: interior node) + kOwn for its first member, w index among the
// groups with more than two members

template <int N>
struct FlatGeo {
    static constexpr int n1 = N + 1, NP = n1 * n1, NI = (N - 1) * (N - 1), NB = NP - NI;
    static constexpr int EPB = NP >= 64 ? 1 : 64 / NP;
    static constexpr int SLOTS = EPB * NP, BLOCK = (SLOTS + 63) / 64 * 64;
};

template <typename T>
struct FlatArgs {
    const T *op;          // operand: interior nodes, and boundary nodes when nothing is pending
    const T *f0in;        // stage: post-collision state (interior)
    T *out;               // result: interior nodes (filter: all; may be op)
    T *y;                 // first stage: post-collision state
    T *opb;               // stage: the operand's boundary nodes are stored here
    // pending assembly of the operand's boundary nodes: pca f0 + pcb fk + pcc L
    const T *pf0, *pfk, *rin, *rhop;
    T pca, pcb, pcc;
    int pend;
    T *rout;              // contributions of this stage
    const T *rho;         // stage: density at the collision
    T *rhoc;              // first stage: written here
    const T *Gm, *invw, *invMb, *D, *F, *wallu, *Fn;
    const float *dtau;
    const int4 *nodes;
    const int32_t *ftag;
    int64_t E, Gi, QGi, plane, ngp, nmp;
    T dt, omega, tau, rho0, ca, cb, cc, g[3], fsc[9];
    int filter;
};

enum { F_FIRST = 0, F_STAGE = 1, F_FILTER = 2 };

template <int N, typename T, bool DEV, int MODE>
__global__ void __launch_bounds__((FlatGeo<N>::BLOCK)) k_flat(FlatArgs<T> A)
{
    using G = FlatGeo<N>;
    constexpr int Q = 9, n1 = G::n1, NP = G::NP, NI = G::NI, EPB = G::EPB;
    constexpr bool DIF = std::is_same<T, float>::value;
    __shared__ T pl[Q][G::SLOTS];
    __shared__ T sD[n1 * n1], sF[MODE == F_STAGE ? 1 : n1 * n1];
    const int tid = threadIdx.x, le = EPB == 1 ? 0 : tid / NP, p = tid - le * NP;
    const int64_t nblk = (A.E + EPB - 1) / EPB, eb = xcd_block(nblk);
    if (eb >= nblk) return;  // whole workgroup
    const int64_t e = eb * EPB + le;
    const bool valid = tid < G::SLOTS && e < A.E;
    const int4 nd = valid ? A.nodes[e * NP + p] : int4{0, 0, 0, 0};
    for (int q = tid; q < n1 * n1; q += G::BLOCK) {
        sD[q] = A.D[q];
        if constexpr (MODE != F_STAGE) sF[q] = A.F[q];
    }
    const int i = p % n1, j = (p / n1) % n1;
    T Gr[2][2] = {};
    uint32_t wcode = 0;
    if (MODE != F_FILTER && valid) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 2; ++q) Gr[m][q] = A.Gm[(e * 4 + m * 2 + q) * NP + p];
        // wall faces through the node: 8 bits per direction, tag and bit 7 for r_m = +1
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int ix = m == 0 ? i : j;
            const uint32_t tag = (ix == 0 || ix == N) ? (uint32_t)A.ftag[e * 4 + 2 * m + (ix == N ? 1 : 0)] : 0u;
            if (tag) wcode |= (tag | (ix == N ? 0x80u : 0u)) << (8 * m);
        }
    }
    const int nm = nd.z & (kOwn - 1);
    const bool inner = nm == 0, own = valid && (inner || (nd.z & kOwn));
    const int64_t gix = inner ? e * NI + nd.x : A.Gi + nd.x;
    const SIdx si = inner ? sidx_interior(e, nd.x, Q, NI) : sidx_group(nd.x, Q, A.QGi);
    T Fv[3] = {T(0), T(0), T(0)};
    if (A.Fn && valid) {
#pragma unroll
        for (int c = 0; c < 2; ++c) Fv[c] = A.Fn[3 * gix + c];
    }
    // F* of velocity a at the node
    auto fstar = [&](auto AA, T rho) {
        constexpr int a = decltype(AA)::value;
        T L = A.fsc[a] * rho;
        if (A.Fn) L += T(3.0 * lat_t<2, Q>(a)) * edot<lat_e<2, Q>(a, 0), lat_e<2, Q>(a, 1), 0>(Fv[0], Fv[1], T(0));
        return L;
    };
    T v[Q] = {}, f0[MODE == F_STAGE ? Q : 1] = {};
    T invw = 0, rho = 0;
    if (valid && (inner || !A.pend)) {
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            v[a] = A.op[si.base + a * si.stride];
        });
        if (MODE == F_STAGE && inner)
            static_for<0, Q>([&](auto AA) {
                constexpr int a = decltype(AA)::value;
                f0[MODE == F_STAGE ? a : 0] = A.f0in[si.base + a * si.stride];
            });
        if (inner && MODE != F_FILTER) {
            invw = A.invw[gix];
            if constexpr (MODE == F_STAGE) rho = A.rho[gix];
        }
    } else if (valid) {
        // the node's members in ascending order, then the update of the last stage
        const T *r = A.rin + nd.x, *x = A.rin + 2 * A.ngp + nd.w;
        // (all loads first; a member's block is skipped where no node has it)
        T s[Q] = {}, s1[Q] = {}, s2[Q] = {}, s3[Q] = {}, b0[Q], bk[Q];
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            if constexpr (a > 0) s[a] = r[a * A.plane];
            b0[a] = A.pf0[si.base + a * si.stride];
            bk[a] = A.pfk[si.base + a * si.stride];
        });
        const T iM = A.invMb[nd.x], rg = A.rhop[gix];
        auto member = [&](bool has, const T *q, T (&d)[Q]) {
            if (has)
                static_for<1, Q>([&](auto AA) {
                    constexpr int a = decltype(AA)::value;
                    d[a] = q[a * A.plane];
                });
        };
        member(nm > 1, r + A.ngp, s1);
        member(nm > 2, x, s2);
        member(nm > 3, x + A.nmp, s3);
        static_for<1, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            s[a] = ((s[a] + s1[a]) + s2[a]) + s3[a];
        });
        for (int t = 4; t < nm; ++t)
            static_for<1, Q>([&](auto AA) {
                constexpr int a = decltype(AA)::value;
                s[a] += x[a * A.plane + (t - 2) * A.nmp];
            });
        static_for<0, Q>([&](auto AA) {
            constexpr int a = decltype(AA)::value;
            v[a] = rk_combine(A.pca, A.pcb, A.pcc, b0[a], bk[a], s[a] * iM + fstar(AA, rg), 1);
            if (MODE == F_STAGE && own) A.opb[si.base + a * si.stride] = v[a];
        });
    }
    const int base = le * NP, rowr = base + n1 * j, rows = base + i;
    auto fill = [&] {
        if (tid < G::SLOTS)
            static_for<0, Q>([&](auto AA) {
                constexpr int a = decltype(AA)::value;
                pl[a][tid] = v[a];
            });
    };
    if constexpr (MODE != F_STAGE) {
        if (A.filter) {
            // explicit modal filter (Sec. 2.2.3), one direction per pass
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                if (m) __syncthreads();
                fill();
                __syncthreads();
                const int ir = m == 0 ? i : j, row = m == 0 ? rowr : rows, str = m == 0 ? 1 : n1;
                if (tid < G::SLOTS)
                    static_for<0, Q>([&](auto AA) {
                        constexpr int a = decltype(AA)::value;
                        const T x = v[a];
                        T t = 0;
#pragma unroll
                        for (int q = 0; q < n1; ++q) {
                            if constexpr (DIF) t += sF[ir * n1 + q] * (pl[a][row + str * q] - x);
                            else t += sF[ir * n1 + q] * pl[a][row + str * q];
                        }
                        v[a] = DIF ? t + x : t;
                    });
            }
        }
        if constexpr (MODE == F_FILTER) {
            if (own)
                static_for<0, Q>([&](auto AA) {
                    constexpr int a = decltype(AA)::value;
                    A.out[si.base + a * si.stride] = v[a];
                });
            return;
        }
    }
    if constexpr (MODE == F_FIRST) {
        if (valid) {
            const T om = A.dtau ? T(1) / (A.tau + T(A.dtau[gix]) + T(0.5)) : A.omega;
            collide_node<2, Q, T, DEV>(v, A.rho0, om, A.dt, A.g, rho, Fv, A.Fn != nullptr);
            if (own) {
                static_for<0, Q>([&](auto AA) {
                    constexpr int a = decltype(AA)::value;
                    A.y[si.base + a * si.stride] = v[a];
                });
                A.rhoc[gix] = rho;
            }
        }
        __syncthreads();  // the filter's reads of the planes are done
    }
    fill();
    __syncthreads();
    if (!valid) return;
    T Di[n1], Dj[n1];
#pragma unroll
    for (int c = 0; c < n1; ++c) {
        Di[c] = sD[i * n1 + c];
        Dj[c] = sD[j * n1 + c];
    }
    static_for<0, Q>([&](auto AA) {
        constexpr int a = decltype(AA)::value;
        T rt = stream_volume<2, N, Q, a, DIF>(pl[a], v[a], Di, Dj, Dj, Gr, rowr, rows, 0);
        if (wcode) wall_flux<2, N, Q, a>(rt, v[a], v[lat_opp<2, Q>(a)], Gr, wcode, A.wallu, A.rho0);
        if (inner) {
            T f;
            if constexpr (MODE == F_STAGE) f = f0[a];
            else f = v[a];
            A.out[si.base + a * si.stride] = rk_combine(A.ca, A.cb, A.cc, f, v[a], rt * invw + fstar(AA, rho), 1);
        } else if constexpr (a > 0) {
            A.rout[a * A.plane + nd.y] = rt;
        }
    });
}

}  // namespace sel
