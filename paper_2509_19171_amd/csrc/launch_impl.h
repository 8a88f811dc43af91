// Launch sequences of the SELBM kernels for one (dim, N, Q, storage) choice.
#pragma once

#include <utility>

#include "kernels_big.h"
#include "kernels_flat.h"
#include "kernels_impl.h"
#include "kernels_mfma.h"
#include "kernels_relax.h"
#include "kernels_stream.h"
#include "ops.h"

namespace sel {

#define SEL_LAUNCH_CHECK()                                                                  \
    do {                                                                                    \
        hipError_t err_ = hipGetLastError();                                                \
        if (err_ != hipSuccess) {                                                           \
            set_error(std::string("kernel launch failed: ") + hipGetErrorString(err_));    \
            return SEL_EDEVICE;                                                             \
        }                                                                                   \
    } while (0)

template <int DIM, int N, int Q, typename T, bool DEV>
struct Impl {
    using GG = Geo<DIM, N>;
    static constexpr int NP = GG::NP, NI = GG::NI, NB = GG::NB, EPB = GG::EPB;
    // later-stage element kernel with matrix-core contractions (kernels_mfma.h)
    static constexpr bool kMfma = std::is_same<T, float>::value && DEV && DIM == 3 && N == 7;
    // 3D orders whose element has more nodes than a workgroup has threads
    // (kernels_big.h): several nodes per thread
    static constexpr bool kBig = DIM == 3 && NP > 1024;

    static T *st(sel_sim *s, int i) { return static_cast<T *>(s->f[i]); }
    static int64_t nblk(sel_sim *s) { return (s->E + EPB - 1) / EPB; }

    static NodeMap nodemap(sel_sim *s)
    {
        NodeMap M;
        M.pcode = s->pcode;
        M.bmap = s->bmap;
        M.bown = s->bown;
        M.E = s->E;
        M.Gi = s->Gi;
        M.QGi = (int64_t)Q * s->Gi;
        M.NP = NP;
        M.NI = NI;
        M.NB = NB;
        M.Q = Q;
        return M;
    }

    static StageArgs<T> stage_args(sel_sim *s)
    {
        StageArgs<T> A{};
        A.Gm = static_cast<const T *>(s->Gm);
        A.invw = static_cast<const T *>(s->invw);
        A.D = static_cast<const T *>(s->tabD);
        A.F = static_cast<const T *>(s->tabF);
        A.pcode = s->pcode;
        A.bmap = s->bmap;
        A.bpos = s->bpos;
        A.ftag = s->ftag;
        A.bown = s->bown;
        A.wallu = static_cast<const T *>(s->wallu);
        A.nbr = s->nbr;
        A.E = s->E;
        A.nblk = nblk(s);
        A.Gi = s->Gi;
        A.QGi = (int64_t)Q * s->Gi;
        A.dt = T(s->p.dt);
        A.omega = T(s->omega);
        A.rho0 = T(s->p.rho0);
        for (int q = 0; q < 3; ++q) A.g[q] = T(q < DIM ? s->p.accel[q] : 0.0);
        for (int a = 0; a < Q; ++a) A.fsc[a] = T(s->fsc[a]);
        A.rtb = static_cast<T *>(s->rtb);
        A.posmap = s->posmap;
        A.plane = s->plane;
        A.rhoc = static_cast<T *>(s->rhoc);
        A.tau = T(s->tau);
        A.dtau = nullptr;
        return A;
    }

    static GroupArgs<T> group_args(sel_sim *s)
    {
        GroupArgs<T> B{};
        B.rtb = static_cast<const T *>(s->rtb);
        B.rhoc = static_cast<const T *>(s->rhoc);
        B.invMb = static_cast<const T *>(s->invMb);
        B.goff = s->goff;
        B.hidx = s->hidx;
        B.ngrp = s->ngrp;
        B.Gi = s->Gi;
        B.QGi = (int64_t)Q * s->Gi;
        B.plane = s->plane;
        B.ngp = s->ngp;
        B.nmp = s->nmp;
        for (int a = 0; a < Q; ++a) B.fsc[a] = T(s->fsc[a]);
        B.nbr = s->nbr;
        B.ftag = s->ftag;
        B.bpos = s->bpos;
        B.Gm = static_cast<const T *>(s->Gm);
        return B;
    }

    // events around a launch when sel_step_timed asked for them
    static int tic(sel_sim *s, int kind, hipEvent_t &b)
    {
        if (!s->timing) return SEL_OK;
        hipEvent_t e0, e1;
        if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return SEL_EDEVICE;
        s->timing->push_back({kind, {e0, e1}});
        b = e1;
        return hipEventRecord(e0, s->stream) == hipSuccess ? SEL_OK : SEL_EDEVICE;
    }
    static int toc(sel_sim *s, hipEvent_t b)
    {
        if (!s->timing) return SEL_OK;
        return hipEventRecord(b, s->stream) == hipSuccess ? SEL_OK : SEL_EDEVICE;
    }

    // Workgroups an element's passes over its velocities are dealt to: small
    // meshes leave most of the chip idle while one workgroup goes through an
    // element's passes in turn: about four workgroups per CU, two of those with
    // more than 40 KB of LDS (Taylor-Green N = 7 FP64, three steps: 4^3 elements
    // 352 -> 290 us, 6^3 403 -> 340; 8^3 N = 12, two per CU already, stays unsplit:
    // 121 us a stage against 132)
    static int split_of(int64_t E, int passes, size_t lds)
    {
        const int64_t n = (lds > 40 * 1024 ? 512 : 1024) / E;
        return n <= 1 ? 1 : n < passes ? (int)n : passes;
    }

    // affine elements (3D): one streaming pass (kernels_stream.h) with the operands of A
    static int launch_stream(sel_sim *s, const StageArgs<T> &A)
    {
        using SG = StreamGeo<N, Q, T>;
        StreamArgs<N, Q, T> S{};
        S.op = A.op;
        S.f0in = A.f0in;
        S.out = A.out;
        S.rtb = A.rtb;
        S.rhoc = A.rhoc;
        S.wallu = A.wallu;
        S.Fn = A.Fn;
        S.bpos = A.bpos;
        S.bmap = A.bmap;
        S.posmap = A.posmap;
        S.ftag = A.ftag;
        S.E = A.E;
        S.QGi = A.QGi;
        S.plane = A.plane;
        S.ca = A.ca;
        S.cb = A.cb;
        S.cc = A.cc;
        S.rho0 = A.rho0;
        S.incr = A.incr;
        S.same = A.f0in == A.op;
        S.tab = static_cast<const T *>(s->tabL);
        S.aff = static_cast<const T *>(s->aff);
        for (int i = 0; i <= N; ++i) S.w[i] = T(s->tab.w[i]);
        int n = 0;
        for (int a = 1; a < Q; ++a) {
            const int b = lat_opp<DIM, Q>(a);
            if (b < a) continue;
            S.pa[n] = a;
            S.pb[n] = b;
            for (int c = 0; c < 3; ++c) S.pe[n][c] = T(lat_e<DIM, Q>(a, c));
            S.pt[n] = T(lat_t<DIM, Q>(a));
            S.pf[n] = A.fsc[a];
            S.body |= A.fsc[a] != T(0);
            ++n;
        }
        hipEvent_t ev = nullptr;
        if (int rc = tic(s, 1, ev)) return rc;
        S.split = split_of(A.E, SG::PASSES, sizeof(T) * SG::UPB * 3 * SG::PL);
        const dim3 grid((unsigned)xcd_grid(A.E * S.split)), block(SG::BLOCK);
        if (s->nwall > 0) {
            hipLaunchKernelGGL((k_stream<N, Q, T, true>), grid, block, 0, s->stream, S);
        } else {
            hipLaunchKernelGGL((k_stream<N, Q, T, false>), grid, block, 0, s->stream, S);
        }
        SEL_LAUNCH_CHECK();
        return toc(s, ev);
    }

    // 3D: the state S (filtered first when `filter`) collided into out, or with
    // collide = false only filtered
    static int launch_relax(sel_sim *s, const T *S, T *out, bool filter, bool collide, const float *dtau, bool force)
    {
        using RG = RelaxGeo<N, Q, T>;
        RelaxArgs<T> A{};
        A.op = S;
        A.out = out;
        A.rhoc = static_cast<T *>(s->rhoc);
        A.tab = static_cast<const T *>(s->tabL) + LineTab<N + 1>::size;
        A.Fn = force ? static_cast<const T *>(s->Fn) : nullptr;
        A.dtau = dtau;
        A.bpos = s->bpos;
        A.bmap = s->bmap;
        A.bown = s->bown;
        A.E = s->E;
        A.Gi = s->Gi;
        A.Gtot = s->Gtot;
        A.QGi = (int64_t)Q * s->Gi;
        A.dt = T(s->p.dt);
        A.omega = T(s->omega);
        A.tau = T(s->tau);
        A.rho0 = T(s->p.rho0);
        for (int q = 0; q < 3; ++q) A.g[q] = T(s->p.accel[q]);
        hipEvent_t ev = nullptr;
        if (int rc = tic(s, collide ? 0 : 3, ev)) return rc;
        const int64_t nb = (s->E + RG::EPB - 1) / RG::EPB;
        if (filter && RG::FUSED) {
            const dim3 grid((unsigned)xcd_grid(nb)), block(RG::BLOCK);
            if constexpr (RG::FUSED) {
                if (collide) hipLaunchKernelGGL((k_relax<N, Q, T, DEV, true>), grid, block, 0, s->stream, A);
                else hipLaunchKernelGGL((k_relax<N, Q, T, DEV, false>), grid, block, 0, s->stream, A);
            }
        } else {
            if constexpr (!RG::FUSED) {
                if (filter) {
                    using FG = FilterGeo<N, Q, T>;
                    A.split = split_of(s->E, (Q + FG::UPB - 1) / FG::UPB, sizeof(T) * FG::UPB * StreamGeo<N, Q, T>::PL);
                    hipLaunchKernelGGL((k_filter<N, Q, T>), dim3((unsigned)xcd_grid(s->E * A.split)),
                                       dim3(FG::BLOCK), 0, s->stream, A);
                    A.op = A.out;
                }
            }
            if (collide)
                hipLaunchKernelGGL((k_collide<N, Q, T, DEV>), dim3((unsigned)((s->Gtot + 255) / 256)), dim3(256), 0,
                                   s->stream, A);
        }
        SEL_LAUNCH_CHECK();
        return toc(s, ev);
    }

    template <int MODE>
    static int launch_stage(sel_sim *s, const StageArgs<T> &A)
    {
        static_assert(DIM == 2 || MODE != M_FILTER, "3D: launch_relax");
        if constexpr (DIM == 3 && MODE == M_STAGE23) {
            if (s->aff) return launch_stream(s, A);
        }
        dim3 grid((unsigned)xcd_grid(A.nblk)), block(GG::BLOCK);
        hipEvent_t ev = nullptr;
        const int kind = (MODE == M_STAGE1) ? 0 : (MODE == M_STAGE23) ? 1 : 3;
        if constexpr (kBig) {
            if (A.nbr) {
                set_error("the discontinuous coupling takes one thread per element node: 3D orders with at most 1024 nodes (N <= 9)");
                return SEL_EUNSUPPORTED;
            }
            if (int rc = tic(s, kind, ev)) return rc;
            bool fn = false;
            if constexpr (MODE == M_STAGE23) {
                fn = A.Fn != nullptr;
                if (fn)
                    hipLaunchKernelGGL((k_stage_big<N, Q, T, MODE, true>), grid, dim3(BigGeo<N>::BLOCK), 0, s->stream, A);
            }
            if (!fn)
                hipLaunchKernelGGL((k_stage_big<N, Q, T, MODE>), grid, dim3(BigGeo<N>::BLOCK), 0, s->stream, A);
        } else {
            if (int rc = tic(s, kind, ev)) return rc;
            // element contributions under the discontinuous coupling carry the
            // interface flux themselves; in the stages it is added by the
            // assembly (k_group_split), where every element-boundary node is a group
            bool dg = false;
            if constexpr (MODE == M_LOCAL) {
                dg = A.nbr != nullptr;
                if (dg) {
                    hipLaunchKernelGGL((k_stage<DIM, N, Q, T, DEV, MODE, true>), grid, block, 0, s->stream, A);
                }
            }
            if (!dg) {
                // FP32 3D order 7, later stages: vector loads and matrix-core contractions
                if constexpr (kMfma && MODE == M_STAGE23) {
                    if (A.Fn) hipLaunchKernelGGL((k_stage23_mf<Q, true>), grid, block, 0, s->stream, A);
                    else hipLaunchKernelGGL((k_stage23_mf<Q>), grid, block, 0, s->stream, A);
                } else {
                    bool fn = false;
                    if constexpr ((MODE == M_STAGE1 && DIM == 2) || MODE == M_STAGE23) {
                        fn = A.Fn != nullptr;
                        if (fn)
                            hipLaunchKernelGGL((k_stage<DIM, N, Q, T, DEV, MODE, false, true>), grid, block, 0,
                                               s->stream, A);
                    }
                    if (!fn) hipLaunchKernelGGL((k_stage<DIM, N, Q, T, DEV, MODE>), grid, block, 0, s->stream, A);
                }
            }
        }
        SEL_LAUNCH_CHECK();
        return toc(s, ev);
    }

    // Wavefronts that share 64 groups of the assembly. Four hide more latency as
    // long as all their workgroups are resident at once (8 per CU in FP32, 5 in
    // FP64), two have fewer to run after that, until they need another round
    // themselves (8 per CU in FP32, 5 or, D3Q27, 4 in FP64): then four are ahead
    // again, in FP32 where that round is less than a third full and few went
    // before. us with 2 and 4: FP32 D3Q27 61 k groups 15.0 and 12.2, 127 k 17.7 and
    // 15.1, 152 k 19.1 and 21.2, 219 k 23.1 and 24.9, 292 k 34.9 and 31.6, 520 k 53.6 and
    // 56.0; FP64 D3Q27 65 k 17.6 and 16.4, 97 k 26.4 and 29.9, 152 k 39.5 and 38.1. With
    // the discontinuous coupling each of them looks up the faces: 33 k groups 9.6 and
    // 9.1, 152 k 17.4 and 19.5.
    static int assembly_split(int64_t n, bool dg)
    {
        constexpr int64_t cu = 256;
        if (dg) return n <= 144 * cu ? 4 : 2;
        constexpr int64_t r4 = 64 * cu * (sizeof(T) == 4 ? 8 : 5);
        constexpr int64_t r2 = 128 * cu * (sizeof(T) == 4 ? 8 : Q == 27 ? 4 : 5);
        if (n <= r4) return 4;
        if (sizeof(T) == 8) return n > r2 ? 4 : 2;
        return Q != 9 && n > r2 && n < 3 * r2 && 3 * (n % r2) < r2 ? 4 : 2;
    }

    static int launch_group(sel_sim *s, const GroupArgs<T> &B)
    {
        if (s->ngrp == 0) return SEL_OK;
        dim3 block(256);
        hipEvent_t ev = nullptr;
        if (int rc = tic(s, 2, ev)) return rc;
        // the discontinuous coupling adds its interface flux here
        const int split = assembly_split(s->ngrp, B.nbr != nullptr);
        const dim3 grid((unsigned)xcd_grid((s->ngrp * split + 255) / 256));
        auto launch = [&](auto FN) {
            constexpr bool fn = decltype(FN)::value;
            if (B.nbr && split == 4) {
                hipLaunchKernelGGL((k_group_split<Q, T, 4, N, fn>), grid, block, 0, s->stream, B);
            } else if (B.nbr) {
                hipLaunchKernelGGL((k_group_split<Q, T, 2, N, fn>), grid, block, 0, s->stream, B);
            } else if (split == 4) {
                hipLaunchKernelGGL((k_group_split<Q, T, 4, 0, fn>), grid, block, 0, s->stream, B);
            } else {
                hipLaunchKernelGGL((k_group_split<Q, T, 2, 0, fn>), grid, block, 0, s->stream, B);
            }
        };
        if (B.Fn) launch(std::true_type{});
        else launch(std::false_type{});
        SEL_LAUNCH_CHECK();
        return toc(s, ev);
    }

    static int geometry(sel_sim *s)
    {
        const int64_t nb = nblk(s);
        if constexpr (kBig) {
            hipLaunchKernelGGL((k_geom_big<N, T>), dim3((unsigned)nb), dim3(BigGeo<N>::BLOCK), 0, s->stream, s->xyz,
                               s->geoD, s->geoW, s->wJ, s->J, static_cast<T *>(s->Gm), s->flag, s->E);
        } else {
            hipLaunchKernelGGL((k_geom<DIM, N, T>), dim3((unsigned)nb), dim3(GG::BLOCK), 0, s->stream, s->xyz,
                               s->geoD, s->geoW, s->wJ, s->J, static_cast<T *>(s->Gm), s->flag, s->E, nb);
        }
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    static int mass(sel_sim *s)
    {
        const int64_t nl = s->E * NP;
        hipLaunchKernelGGL((k_mass_int<T>), dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, s->stream, s->wJ,
                           s->pcode, static_cast<T *>(s->invw), s->E, NP, NI);
        SEL_LAUNCH_CHECK();
        if (s->ngrp > 0) {
            hipLaunchKernelGGL((k_mass_grp<T>), dim3((unsigned)((s->ngrp + 255) / 256)), dim3(256), 0, s->stream,
                               s->wJ, s->bpos, s->goff, s->gmem, static_cast<T *>(s->invMb), s->ngrp, NP, NB);
            SEL_LAUNCH_CHECK();
        }
        return SEL_OK;
    }

    static int init(sel_sim *s, const double *d_rho, const double *d_u)
    {
        const int64_t nl = s->E * NP;
        hipLaunchKernelGGL((k_init<DIM, Q, T, DEV>), dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, s->stream,
                           nodemap(s), d_rho, d_u, st(s, s->cur), s->p.rho0, s->p.dt, s->p.accel[0],
                           s->p.accel[1], DIM == 3 ? s->p.accel[2] : 0.0);
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    // mirrored tables of the line operators (LineTab): the derivative matrix,
    // then the modal filter minus the identity
    static int line_tables(const Tables &t, double *out)
    {
        constexpr int n1 = N + 1;
        double M[n1 * n1];
        line_tab<n1>(t.D, out);
        for (int q = 0; q < n1 * n1; ++q) M[q] = t.F[q] - (q % (n1 + 1) == 0 ? 1.0 : 0.0);
        line_tab<n1>(M, out + LineTab<n1>::size);
        return 2 * LineTab<n1>::size;
    }

    // one time step: collide (and filter the previous step's result) ->
    // SSPRK3 streaming with F* and the wall flux; the filter of this step is
    // applied by the next step's first stage, or at the end of the call.
    // per-node force density (added to rho g): fill from FP64 [E][np][dim]
    static int set_force(sel_sim *s, const double *d_F)
    {
        const int64_t nl = s->E * NP;
        hipLaunchKernelGGL((k_force_set<T>), dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, s->stream, nodemap(s),
                           d_F, DIM, static_cast<T *>(s->Fn));
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    // One element pass and its assembly: out = ca f0 + cb fk + cc L(fk).
    static int stage_pass(sel_sim *s, StageArgs<T> &A, GroupArgs<T> &B, const T *fk, const T *f0, T *out,
                          double ca, double cb, double cc)
    {
        A.op = fk;
        A.f0in = f0;
        A.out = out;
        A.ca = T(ca);
        A.cb = T(cb);
        A.cc = T(cc);
        if (int rc = launch_stage<M_STAGE23>(s, A)) return rc;
        B.f0 = f0;
        B.fk = fk;
        B.out = out;
        B.ca = T(ca);
        B.cb = T(cb);
        B.cc = T(cc);
        return launch_group(s, B);
    }

    // The first stage of a 3D mesh that is not streamed by k_stream, and has the
    // continuous coupling and no force per node, in one kernel (M_STAGE1)
    // instead of a collision pass and a streaming pass, or three passes with a filter
    // pending: the post-collision state is not read back. With few elements it is
    // the launch that counts; with many the separate kernels hold more
    // wavefronts, so that FP32 keeps them, while FP64 streams a chunk of
    // velocities at a time either way. Per step, us, separate and joined, without a
    // filter: FP64 D3Q27 N = 5 1024 elements 228 and 214, 4096 847 and 819, N = 7 20,480
    // 9030 and 8640, N = 8 1024 812 and 855 (it spills); N = 4 1024 FP64 134 and 124, FP32
    // 117 and 108, 16^3 FP64 365 and 386, FP32 220 and 225; N = 7 12^3 FP32 325 and 335.
    // Filtered: FP64 N = 7 8^3 199 and 187, 20,480 elements 9860 and 9420, N = 5 1024 243 and
    // 235, 16^3 777 and 802; FP32 N = 5 1024 131 and 132.
    // Orders up to 3 take the filter along (N = 2 30^3 D3Q19 FP32 277 and 256, N = 3
    // 24^3 FP64 527 and 514).
    static constexpr bool kFirst = DIM == 2 || (!kBig && (sizeof(T) == 8 ? !(N == 8 && Q == 27) : N <= 4));
    static bool first_stage(const sel_sim *s, bool pending)
    {
        if (DIM != 3 || !kFirst || s->aff || s->nbr || s->force_on) return false;
        const int64_t nodes = s->E * NP;
        if (!pending) return (sizeof(T) == 8 && N >= 5) || nodes <= 200000;
        if (N <= kFusedFilter3 || N >= 7) return true;
        return nodes <= (N == 4 ? 160000 : N == 5 ? 225000 : 400000);
    }

    // First stage: filter (when pending) and collide the state S into the
    // post-collision state y = F0, then FA = y + cc L(y), by a streaming pass like
    // the later stages' or in the same kernel (first_stage; 2D: with the
    // continuous coupling, whose shared nodes need no value of another element).
    static int stage_one(sel_sim *s, StageArgs<T> &A, GroupArgs<T> &B, const T *S, T *F0, T *FA, double cc,
                         bool pending)
    {
        if constexpr (DIM == 3) {
            if constexpr (kFirst) {
                if (first_stage(s, pending)) {
                    T *H = st(s, s->cur ^ 1);  // free until the second stage
                    const bool before = pending && N > kFusedFilter3;
                    if (before)
                        if (int rc = launch_relax(s, S, H, true, false, nullptr, false)) return rc;
                    A.op = before ? H : S;
                    A.f0out = F0;
                    A.out = FA;
                    A.ca = T(0);
                    A.cb = T(1);
                    A.cc = T(cc);
                    A.filter = pending && !before;
                    if (int rc = launch_stage<M_STAGE1>(s, A)) return rc;
                    B.f0 = B.fk = F0;
                    B.out = FA;
                    B.ca = T(0);
                    B.cb = T(1);
                    B.cc = T(cc);
                    return launch_group(s, B);
                }
            }
            if (int rc = launch_relax(s, S, F0, pending, true, A.dtau, s->force_on)) return rc;
            return stage_pass(s, A, B, F0, F0, FA, 0.0, 1.0, cc);
        } else {
            A.op = S;
            A.f0out = F0;
            A.filter = pending ? 1 : 0;
            A.collide_only = s->nbr != nullptr;
            A.out = FA;
            A.ca = T(0);
            A.cb = T(1);
            A.cc = T(cc);
            if (int rc = launch_stage<M_STAGE1>(s, A)) return rc;
            if (s->nbr) return stage_pass(s, A, B, F0, F0, FA, 0.0, 1.0, cc);
            B.f0 = B.fk = F0;
            B.out = FA;
            B.ca = T(0);
            B.cb = T(1);
            B.cc = T(cc);
            return launch_group(s, B);
        }
    }

    // The four printed stage formulas of Sec. 2.2.2 with L applied linearly
    // to their combinations (stage values w1..w3, y the post-collision state):
    //   w1 = y + dt/3 L(y)
    //   w2 = w1 - 3dt/4 (L(y) - L(w1))
    //   w3 = w2 + 2dt/3 (L(y) - L(w1) + L(w2))
    //   y' = w3 - dt/4 (L(y) - L(w1) + L(w2) - L(w3)).
    // Each earlier L is eliminated through the stage that defines it, so every
    // stage is a two-state combination ca f0 + cb fk + cc L(fk) with
    // ca + cb = 1 (exact in exact arithmetic, also for an affine L):
    //   w2 = 9/4 y - 5/4 w1 + 3dt/4 L(w1)
    //   w3 = 8/9 w1 + 1/9 w2 + 2dt/3 L(w2)
    //   y' = 3/8 w2 + 5/8 w3 + dt/4 L(w3).
    // Arrays: S holds the state and then y'; F0 holds y and then w3; FA w1;
    // FB w2.
    static int printed4(sel_sim *s, StageArgs<T> &A, GroupArgs<T> &B, T *S, T *FB, T *F0, T *FA, bool pending)
    {
        const double dt = s->p.dt;
        if (int rc = stage_one(s, A, B, S, F0, FA, dt / 3.0, pending)) return rc;
        if (int rc = stage_pass(s, A, B, FA, F0, FB, 9.0 / 4.0, -5.0 / 4.0, 0.75 * dt)) return rc;
        if (int rc = stage_pass(s, A, B, FB, FA, F0, 8.0 / 9.0, 1.0 / 9.0, 2.0 / 3.0 * dt)) return rc;
        return stage_pass(s, A, B, F0, FB, S, 3.0 / 8.0, 5.0 / 8.0, 0.25 * dt);
    }

    // network increments of the closure for the current state (filtered first
    // when `filter`): features, then inference
    static int closure_increments(sel_sim *s, bool filter)
    {
        // the closure reads the filtered state: its features come from the
        // filtered moment fields
        hipEvent_t ev = nullptr;
        if (int rc = tic(s, 4, ev)) return rc;
        if (int rc = features(s, s->cl_X, 1, filter ? 1 : 0)) return rc;
        if (int rc = toc(s, ev)) return rc;
        if (int rc = tic(s, 5, ev)) return rc;
        if (int rc = launch_mlp_infer(s)) return rc;
        return toc(s, ev);
    }

    // 2D, one kernel per stage (kernels_flat.h). Arrays: X the state, whose
    // interior the first stage overwrites with its stage value and the last one
    // with the result; Y the post-collision state; W = f[cur^1] the second stage
    // value; Z the printed stages' third. A stage's boundary values are pending
    // (in its contributions, to be combined from the two states f0 and fk) until
    // the next kernel has assembled them, so no kernel may write the boundary
    // part of those two: with SSPRK3, where Y is one of them, it alternates
    // between f[2] and f[3]. With the discontinuous coupling the assembly, which
    // looks across the faces, runs on its own before the next kernel.
    static int step_flat(sel_sim *s, int64_t nsteps)
    {
        using FG = FlatGeo<N>;
        const double dt = s->p.dt;
        const bool filt = s->p.filter_type != SEL_FILTER_NONE, printed = s->p.rk == SEL_RK_PRINTED4;
        GroupArgs<T> B = group_args(s);
        FlatArgs<T> A{};
        A.Gm = static_cast<const T *>(s->Gm);
        A.invw = static_cast<const T *>(s->invw);
        A.invMb = static_cast<const T *>(s->invMb);
        A.D = static_cast<const T *>(s->tabD);
        A.F = static_cast<const T *>(s->tabF);
        A.wallu = static_cast<const T *>(s->wallu);
        A.Fn = s->force_on ? static_cast<const T *>(s->Fn) : nullptr;
        A.nodes = s->nodes;
        A.ftag = s->ftag;
        A.E = s->E;
        A.Gi = s->Gi;
        A.QGi = (int64_t)Q * s->Gi;
        A.plane = s->plane;
        A.ngp = s->ngp;
        A.nmp = s->nmp;
        A.dt = T(dt);
        A.omega = T(s->omega);
        A.tau = T(s->tau);
        A.rho0 = T(s->p.rho0);
        for (int q = 0; q < 2; ++q) A.g[q] = T(s->p.accel[q]);
        for (int a = 0; a < Q; ++a) A.fsc[a] = T(s->fsc[a]);
        B.Fn = A.Fn;
        B.incr = 1;
        T *rt[2] = {static_cast<T *>(s->rtb), static_cast<T *>(s->rtb2)};
        T *rh[2] = {static_cast<T *>(s->rhoc), static_cast<T *>(s->rhoc2)};
        int kt = 0, kr = 0;  // buffers of the last contributions and densities
        T *X = st(s, s->cur), *W = st(s, s->cur ^ 1), *Y = st(s, 2), *Z = st(s, 3);
        const dim3 grid((unsigned)xcd_grid((s->E + FG::EPB - 1) / FG::EPB)), block(FG::BLOCK);
        auto launch = [&](auto MODE, int kind) -> int {
            constexpr int mode = decltype(MODE)::value;
            A.rin = rt[kt];
            A.rout = rt[kt ^ 1];
            A.rhop = A.rho = rh[kr];
            A.rhoc = rh[kr ^ 1];
            hipEvent_t ev = nullptr;
            if (int rc = tic(s, kind, ev)) return rc;
            hipLaunchKernelGGL((k_flat<N, T, DEV, mode>), grid, block, 0, s->stream, A);
            SEL_LAUNCH_CHECK();
            if (mode != F_FILTER) kt ^= 1;
            if (mode == F_FIRST) kr ^= 1;
            return toc(s, ev);
        };
        // what the boundary nodes of the last result are combined from
        auto pending = [&](const T *f0, const T *fk, double ca, double cb, double cc) {
            A.pf0 = f0;
            A.pfk = fk;
            A.pca = T(ca);
            A.pcb = T(cb);
            A.pcc = T(cc);
            A.pend = 1;
        };
        auto assemble = [&](T *out) -> int {
            B.rtb = rt[kt];
            B.rhoc = rh[kr];
            B.f0 = A.pf0;
            B.fk = A.pfk;
            B.out = out;
            B.ca = A.pca;
            B.cb = A.pcb;
            B.cc = A.pcc;
            A.pend = 0;
            return launch_group(s, B);
        };
        // out = ca f0 + cb fk + cc L(fk), fk pending from before
        auto stage = [&](T *fk, const T *f0, T *out, double ca, double cb, double cc) -> int {
            if (s->nbr)
                if (int rc = assemble(fk)) return rc;
            A.op = A.opb = fk;
            A.f0in = f0;
            A.out = out;
            A.ca = T(ca);
            A.cb = T(cb);
            A.cc = T(cc);
            if (int rc = launch(std::integral_constant<int, F_STAGE>{}, 1)) return rc;
            pending(f0, fk, ca, cb, cc);
            return SEL_OK;
        };
        A.filter = 0;
        for (int64_t n = 0; n < nsteps; ++n) {
            A.dtau = nullptr;
            // the features read the state: it is assembled first
            if (A.pend && (s->nbr || s->closure_on))
                if (int rc = assemble(X)) return rc;
            if (s->closure_on) {
                if (int rc = closure_increments(s, A.filter != 0)) return rc;
                A.dtau = s->cl_dtau;
            }
            if (!printed && A.pend) std::swap(Y, Z);
            const double c1 = printed ? dt / 3.0 : dt;
            A.op = X;
            A.out = X;
            A.y = Y;
            A.ca = T(0);
            A.cb = T(1);
            A.cc = T(c1);
            if (int rc = launch(std::integral_constant<int, F_FIRST>{}, 0)) return rc;
            pending(Y, Y, 0.0, 1.0, c1);
            if (printed) {
                if (int rc = stage(X, Y, W, 9.0 / 4.0, -5.0 / 4.0, 0.75 * dt)) return rc;
                if (int rc = stage(W, X, Z, 8.0 / 9.0, 1.0 / 9.0, 2.0 / 3.0 * dt)) return rc;
                if (int rc = stage(Z, W, X, 3.0 / 8.0, 5.0 / 8.0, 0.25 * dt)) return rc;
            } else {
                if (int rc = stage(X, Y, W, 0.75, 0.25, 0.25 * dt)) return rc;
                if (int rc = stage(W, Y, X, 1.0 / 3.0, 2.0 / 3.0, 2.0 / 3.0 * dt)) return rc;
            }
            A.filter = filt ? 1 : 0;
            s->time += dt;
            s->nstep += 1;
        }
        if (!filt || s->nbr)
            if (int rc = assemble(X)) return rc;
        if (!filt) return SEL_OK;
        // in place: a node's interior value is read by its own thread alone, and its
        // boundary value comes from the two states it is pending on, neither of
        // them X (discontinuous coupling: is the thread's own as well). The state
        // keeps its array from call to call, so a captured call (or a sequence of
        // them) replays from its own result.
        A.op = A.out = X;
        return launch(std::integral_constant<int, F_FILTER>{}, 3);
    }

    static int step(sel_sim *s, int64_t nsteps)
    {
        if (nsteps <= 0) return SEL_OK;
        if constexpr (DIM == 2) {
            if (s->nodes) return step_flat(s, nsteps);
        }
        const double dt = s->p.dt;
        const bool filt = s->p.filter_type != SEL_FILTER_NONE;
        StageArgs<T> A = stage_args(s);
        GroupArgs<T> B = group_args(s);
        A.incr = 1;  // SSPRK weights sum to one
        B.incr = 1;
        A.Fn = B.Fn = s->force_on ? static_cast<const T *>(s->Fn) : nullptr;
        T *F0 = st(s, 2), *FA = st(s, 3);
        bool pending = false;
        for (int64_t n = 0; n < nsteps; ++n) {
            if (s->closure_on) {
                if (int rc = closure_increments(s, pending)) return rc;
                A.dtau = s->cl_dtau;
            } else {
                A.dtau = nullptr;
            }
            T *S = st(s, s->cur), *FB = st(s, s->cur ^ 1);
            if (s->p.rk == SEL_RK_PRINTED4) {
                if (int rc = printed4(s, A, B, S, FB, F0, FA, pending)) return rc;
                pending = filt;
                s->time += dt;
                s->nstep += 1;
                continue;
            }
            // stage 1: f1 = f0 + dt L(f0), f0 = collide(filter(f3_prev) or f-bar)
            if (int rc = stage_one(s, A, B, S, F0, FA, dt, pending)) return rc;
            // stage 2: f2 = 3/4 f0 + 1/4 (f1 + dt L(f1))
            if (int rc = stage_pass(s, A, B, FA, F0, FB, 0.75, 0.25, 0.25 * dt)) return rc;
            // stage 3: f3 = 1/3 f0 + 2/3 (f2 + dt L(f2)), written over the state
            if (int rc = stage_pass(s, A, B, FB, F0, S, 1.0 / 3.0, 2.0 / 3.0, 2.0 / 3.0 * dt)) return rc;
            pending = filt;
            s->time += dt;
            s->nstep += 1;
        }
        if (pending) {
            if constexpr (DIM == 3) {
                if (int rc = launch_relax(s, st(s, s->cur), st(s, s->cur ^ 1), true, false, nullptr, false)) return rc;
            } else {
                A.op = st(s, s->cur);
                A.out = st(s, s->cur ^ 1);
                if (int rc = launch_stage<M_FILTER>(s, A)) return rc;
            }
            s->cur ^= 1;
        }
        return SEL_OK;
    }

    static int moments(sel_sim *s, double *d_rho, double *d_u)
    {
        // (orders of more nodes per element than a workgroup has threads need some
        // elements to have as many loads in flight as with one thread per node: N = 12
        // FP64 64 elements 8.3 and 5.9 us, 125 10.2 and 11.2)
        bool done = false;
        if constexpr (DIM == 3) {
            if (!kBig || s->E > 64) {
                using MG = MomentGeo<N>;
                hipLaunchKernelGGL((k_moments_el<N, Q, T, DEV>), dim3((unsigned)xcd_grid((s->E + MG::EPB - 1) / MG::EPB)),
                                   dim3(MG::BLOCK), 0, s->stream, st(s, s->cur), s->bpos, s->bmap, s->E,
                                   (int64_t)Q * s->Gi, s->p.rho0, d_rho, d_u);
                done = true;
            }
        }
        if (!done) {
            const int64_t nl = s->E * NP;
            hipLaunchKernelGGL((k_moments<DIM, Q, T, DEV>), dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, s->stream,
                               nodemap(s), st(s, s->cur), s->p.rho0, d_rho, d_u);
        }
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    static int reduce(sel_sim *s)
    {
        hipLaunchKernelGGL((k_reduce<DIM, Q, T, DEV>), dim3(s->nred), dim3(256), 0, s->stream, nodemap(s),
                           st(s, s->cur), s->nstate, s->wJ, s->p.rho0, s->red);
        SEL_LAUNCH_CHECK();
        hipLaunchKernelGGL((k_reduce_final<T>), dim3(1), dim3(64), 0, s->stream, s->red, s->nred, s->red + 8 * s->nred);
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    static int scatter(sel_sim *s, int a, const double *d_plane, void *dst, bool sub)
    {
        const int64_t nl = s->E * NP;
        hipLaunchKernelGGL((k_scatter_plane<T>), dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, s->stream,
                           nodemap(s), d_plane, static_cast<T *>(dst), a, sub ? s->toff[a] : 0.0);
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    static int gather(sel_sim *s, int a, const void *src, double *d_plane, bool add)
    {
        const int64_t nl = s->E * NP;
        hipLaunchKernelGGL((k_gather_plane<T>), dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, s->stream,
                           nodemap(s), static_cast<const T *>(src), d_plane, a, add ? s->toff[a] : 0.0);
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    // operator pieces on a state in src (scratch arrays only)
    static int apply(sel_sim *s, int op, void *src_v, void *dst_v, void *local_v)
    {
        T *src = static_cast<T *>(src_v), *dst = static_cast<T *>(dst_v);
        StageArgs<T> A = stage_args(s);
        A.op = src;
        if (op == SEL_OP_RHS || op == SEL_OP_RHS_LOCAL) {
            for (int a = 0; a < Q; ++a) A.fsc[a] = T(0);
            if (hipMemsetAsync(s->rhoc, 0, sizeof(T) * s->Gtot, s->stream) != hipSuccess) return SEL_EDEVICE;
            if (op == SEL_OP_RHS_LOCAL) {
                A.local = static_cast<T *>(local_v);
                return launch_stage<M_LOCAL>(s, A);
            }
            A.f0in = src;
            A.out = dst;
            A.ca = T(0);
            A.cb = T(0);
            A.cc = T(1);
            if (int rc = launch_stage<M_STAGE23>(s, A)) return rc;
            GroupArgs<T> B = group_args(s);
            for (int a = 0; a < Q; ++a) B.fsc[a] = T(0);
            B.f0 = src;
            B.fk = src;
            B.out = dst;
            B.ca = T(0);
            B.cb = T(0);
            B.cc = T(1);
            return launch_group(s, B);
        }
        if constexpr (DIM == 3) {
            if (op == SEL_OP_COLLIDE) return launch_relax(s, src, dst, false, true, nullptr, false);
            if (op == SEL_OP_FILTER) return launch_relax(s, src, dst, true, false, nullptr, false);
            return SEL_EINVAL;
        } else {
        if (op == SEL_OP_COLLIDE) {
            A.f0out = dst;
            A.collide_only = 1;
            A.filter = 0;
            A.ca = A.cb = A.cc = T(0);
            return launch_stage<M_STAGE1>(s, A);
        }
        if (op == SEL_OP_FILTER) {
            A.out = dst;
            return launch_stage<M_FILTER>(s, A);
        }
        return SEL_EINVAL;
        }
    }

    // closure features of the current state: one row per node id
    // (owner_out = 1) or per element node
    static int features(sel_sim *s, float *X, int owner_out, int filter) { return feat(s, X, owner_out, filter, nullptr, 0); }

    // row c of the velocity gradient of the current state, du_c/dx_q per
    // element node [E][np][dim] (FP64, device)
    static int grad_row(sel_sim *s, int c, double *d_out) { return feat(s, nullptr, 0, 0, d_out, c); }

    static int feat(sel_sim *s, float *X, int owner_out, int filter, double *grad, int row)
    {
        if constexpr (kBig) {
            set_error("closure features and velocity gradients take one thread per element node: 3D orders with at most 1024 nodes (N <= 9)");
            return SEL_EUNSUPPORTED;
        } else {
            return feat_launch(s, X, owner_out, filter, grad, row);
        }
    }

    static int feat_launch(sel_sim *s, float *X, int owner_out, int filter, double *grad, int row)
    {
        FeatArgs<T> F{};
        F.grad = grad;
        F.grad_row = row;
        F.f = st(s, s->cur);
        F.F = static_cast<const T *>(s->tabF);
        F.filter = filter;
        F.Gm = static_cast<const T *>(s->Gm);
        F.D = static_cast<const T *>(s->tabD);
        F.wJ = s->wJ;
        F.pcode = s->pcode;
        F.bmap = s->bmap;
        F.bown = s->bown;
        F.X = X;
        F.E = s->E;
        F.nblk = nblk(s);
        F.Gi = s->Gi;
        F.QGi = (int64_t)Q * s->Gi;
        F.rho0 = T(s->p.rho0);
        F.lam = T(s->p.nu * 3.0);
        F.owner_out = owner_out;
        if (grad) {
            hipLaunchKernelGGL((k_features<DIM, N, Q, T, DEV, true>), dim3((unsigned)F.nblk), dim3(GG::BLOCK), 0,
                               s->stream, F);
        } else {
            hipLaunchKernelGGL((k_features<DIM, N, Q, T, DEV>), dim3((unsigned)F.nblk), dim3(GG::BLOCK), 0, s->stream,
                               F);
        }
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    // wJ (u . n) and wJ at every element node, FP64 [2][E][np] (device)
    static int axial_terms(sel_sim *s, const double *n, double *d_out)
    {
        const int64_t nl = s->E * NP;
        hipLaunchKernelGGL((k_axial_terms<DIM, Q, T, DEV>), dim3((unsigned)((nl + 255) / 256)), dim3(256), 0,
                           s->stream, nodemap(s), st(s, s->cur), s->wJ, s->p.rho0, n[0], n[1], DIM == 3 ? n[2] : 0.0,
                           d_out);
        SEL_LAUNCH_CHECK();
        return SEL_OK;
    }

    static const Ops *ops()
    {
        static const Ops o = {geometry, mass, init,    step,     moments,  reduce,   scatter,
                              gather,   apply, features, set_force, grad_row, axial_terms, line_tables};
        return &o;
    }
};

}  // namespace sel
