// z4c_stage.h -- the fused right-hand side / Runge-Kutta stage kernel
// (included by the per-variant translation units z4c_variants_*.hip).
#pragma once
#include "z4c_tile.h"

namespace z4c {
namespace tile {

// Fused right-hand side (+ Runge-Kutta stage) kernel.  Field order: shift,
// conformal metric, Gamma-tilde, lapse, chi, Khat, Theta, At.  Each field's
// right-hand side is finished as soon as its last contribution is known and,
// in a stage, combined with u1/u2 and stored at once; only the new conformal
// metric and At are held back for the det/trace enforcement.  The lapse comes
// before chi, so that the second half of the Ricci tensor, D_i D_j alpha and
// every product with At meet in one place and only nine values wait for it.
// What bounds it: latency (barriers, LDS round trips, HBM) and, with two
// workgroups per CU, about equally HBM traffic.  Measured against the kernel
// with the whole box in LDS and one workgroup per CU (256 points each
// way): RK4 stage 2 of 512 blocks of 16^3 1.371 -> 1.004 ms (3.7 TB/s of HBM
// traffic), RK4 step of 1,024 uneven blocks 18.3 -> 13.1 ms, of 8 x 128^3
// blocks with matter 48.3 -> 28.4 ms (1.8 of it from the tile order).  3 % come
// from the wait for the next field's points before a field's stores (1.036 and
// 13.5 ms without): the stores then drain behind the next field instead of in
// front of it.  Requesting that field later, after the second barrier, takes
// 1.022 ms.
// Non-temporal stores are slower (1.15 ms): the 64-byte row pieces of x
// neighbours no longer meet in L2.  With every load served from one block
// (L2) the 512-block stage takes 0.63 ms.  A loop over tiles (work queue) in
// this kernel keeps per-tile values live across tiles and spills: 1.31 ms.
// Tiles of 8x8x8 (512 threads, one workgroup per CU): 1.04 ms; requesting u1
// and u2 a field earlier: 1.05 ms.
// MON: the constraint monitor of the stage's input state (Sec. 4.1): H,
// M_i, Theta and Z^i formed from the derivatives the stage takes anyway,
// written to a.cons (when not null) and summed per tile into a.partial as
// the constraint kernel does (same per-tile order).
// LOP: lopsided stencils in the advection terms beta^k d_k u; every other
// derivative stays centred.
// NAIVE (right-hand side, float arithmetic only): every staged value is
// rounded to float before the stencil differences (the naive FP32 form).
template <int P, int TX, int TY, int TZ, int WPE, typename R, int MODE, bool GEN, bool MON = false,
          bool LOP = false, bool NAIVE = false>
__global__ void __launch_bounds__(TX *TY *TZ) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
stage_kernel(const StageArgs a)
{
    using D = ColDims<P, TX, TY, TZ>;
    using MZ = MixDimsZ<P, TX, TY, TZ>;
    constexpr int NT = D::NT;
    constexpr bool RK = MODE == MODE_RK;
    // plane part, interior columns, z and y sums of the staged field
    __shared__ double pl[D::NPL];
    __shared__ double zc[D::NZC];
    __shared__ double zs[MZ::NZS];
    __shared__ double ys[MZ::NYS];
    // monitor: per-wave sums of |c| and c^2 of the 8 constraints
    __shared__ double mred[MON ? (NT / 64) * 16 : 1];
    // Long-lived values of each thread in LDS (slot s of thread t at
    // s * NT + t): the Christoffel symbols (conformal metric to chi stage),
    // the shift gradient (shift to chi stage) and, in the latter's place, the
    // At sources (chi to At stage); as many of the 27 as the LDS that the
    // staging leaves at this occupancy holds, the rest in registers.
    constexpr int WG_PER_CU = (4 * WPE * 64) / NT;
    constexpr int SHARE = LDS_PER_CU / LDS_GRANULE / WG_PER_CU * LDS_GRANULE;
    constexpr int STAGED = (D::NPL + D::NZC + MZ::NZS + MZ::NYS) * (int)sizeof(double)
                         + (MON ? (NT / 64) * 16 * (int)sizeof(double) : 8);
    constexpr int SLOT_BUDGET = (SHARE - 64 - STAGED) / (NT * (int)sizeof(R));
    constexpr int NSLOT = SLOT_BUDGET < 27 ? SLOT_BUDGET : 27;
    constexpr int GRANULES = (STAGED + NSLOT * NT * (int)sizeof(R) + LDS_GRANULE - 1) / LDS_GRANULE;
    static_assert(GRANULES * WG_PER_CU * LDS_GRANULE <= LDS_PER_CU, "WG_PER_CU workgroups fit");
    static_assert(NSLOT > 0, "");
    __shared__ R slots[NSLOT * NT];

    {
        const int tile = my_tile();
        const unsigned t = threadIdx.x;
        const unsigned tx = t % TX, ty = (t / TX) % TY, tz = t / (TX * TY);
        R *const sl = slots + t;
        R ex[27 - NSLOT > 0 ? 27 - NSLOT : 1];
        auto put = [&](int s, R v) __attribute__((always_inline)) {
            if (s < NSLOT)
                sl[s * NT] = v;
            else
                ex[s - NSLOT] = v;
        };
        auto get = [&](int s) __attribute__((always_inline)) -> R {
            return s < NSLOT ? sl[s * NT] : ex[s - NSLOT];
        };
        auto GU = [&](int k, int q) __attribute__((always_inline)) { return get(6 * k + q); };
        auto DB = [&](int k, int j) __attribute__((always_inline)) { return get(18 + 3 * k + j); };

        const Tile T = table_entry(a.tiles, tile);
        const z4c_block B = table_entry(a.blocks, T.block);
        const int ng = B.ng;
        const int sy = B.nx + 2 * ng;
        const int sz = sy * (B.ny + 2 * ng);
        const int i = T.i0 + (int)tx, j = T.j0 + (int)ty, k = T.k0 + (int)tz;
        const bool active = i < B.nx && j < B.ny && k < B.nz;
        const int pt = (k + ng) * sz + (j + ng) * sy + (i + ng);
        const unsigned upt8 = 8u * (unsigned)pt;   // byte offset from a uniform field base
        const double *ub = a.u + B.offset;
        const long long fs = B.field_stride;

        double *ob = a.out + B.offset;
        double *u1b = a.u1 ? a.u1 + B.offset : nullptr;
        const double *u2b = a.u2 ? a.u2 + B.offset : nullptr;
        // Values of field f at this point in the u1 and u2 registers.
        struct Old {
            double u1, u2;
        };
        auto old = [&](int f) __attribute__((always_inline)) {
            Old o{0.0, 0.0};
            if constexpr (RK) {
                const long long e = f * fs;
                if (a.rk.read_u1)
                    o.u1 = at(u1b + e, upt8);
                if (a.rk.use_u2 && !a.rk.u2_is_u0)
                    o.u2 = at(u2b + e, upt8);
            }
            return o;
        };
        const Fac<R> F = table_entry(sizeof(R) == sizeof(double) ? (const Fac<R> *)a.fac64
                                                                 : (const Fac<R> *)a.fac32,
                                     T.block);
        FieldTile<P, TX, TY, TZ, GEN> ft;
        ft.setup(a, T, B, t, pl, zc, zs, ys);
        // Stages field FF and requests the next one.
        auto stage = [&](auto FC) __attribute__((always_inline)) {
            constexpr int FF = decltype(FC)::value;
            ft.template stage<FF, next_field<MODE>(FF), NAIVE>();
        };
        ft.st.template prefetch<mixed_field(BETAX)>(BETAX);
        auto staged = [&]() __attribute__((always_inline)) { return ft.centre(); };
        auto centre = [&](int f) __attribute__((always_inline)) {
            return active ? R(at(ub + f * fs, upt8)) : R(0);
        };
        // Values to store: the field (or its right-hand side) and its u1 register.
        struct New {
            double w, n1;
        };
        // Runge-Kutta combination of a field (state u0) with right-hand side kf (FP64).
        auto combine = [&](R kf_r, double u0, const Old &o) __attribute__((always_inline)) {
            const double kf = double(kf_r);
            if constexpr (!RK)
                return New{kf, 0.0};
            const double n1 = o.u1 + a.rk.delta * u0 + a.rk.eps_dt * kf;
            double w = a.rk.g1 * u0 + a.rk.g2 * n1;
            if (a.rk.use_u2)
                w += a.rk.g3 * (a.rk.u2_is_u0 ? u0 : o.u2);
            return New{w + a.rk.beta_dt * kf, n1};
        };
        auto write1 = [&](int f, const New &v) __attribute__((always_inline)) {
            if constexpr (RK)
                if (a.rk.write_u1)
                    at(u1b + f * fs, upt8) = v.n1;
        };
        auto write = [&](int f, const New &v) __attribute__((always_inline)) {
            write1(f, v);
            at(ob + f * fs, upt8) = v.w;
        };

        R g[6];
        sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            g[q] = active ? R(at(ub + (GXX + q) * fs, upt8)) : ((q == 0 || q == 3 || q == 5) ? R(1) : R(0));
        });
        R gi[6];
        {
            const R det = g[0] * (g[3] * g[5] - g[4] * g[4]) - g[1] * (g[1] * g[5] - g[4] * g[2])
                        + g[2] * (g[1] * g[4] - g[3] * g[2]);
            const R id = R(1) / det;
            gi[0] = (g[3] * g[5] - g[4] * g[4]) * id;
            gi[1] = (g[2] * g[4] - g[1] * g[5]) * id;
            gi[2] = (g[1] * g[4] - g[2] * g[3]) * id;
            gi[3] = (g[0] * g[5] - g[2] * g[2]) * id;
            gi[4] = (g[2] * g[1] - g[0] * g[4]) * id;
            gi[5] = (g[0] * g[3] - g[1] * g[1]) * id;
        }
        const R beta[3] = {centre(BETAX), centre(BETAY), centre(BETAZ)};
        const R alpha = active ? R(at(ub + ALPHA * fs, upt8)) : R(1);
        const R pi = R(PI);

        // Derivatives of the staged field; LOP: the lopsided ones in lop.
        R lop[3];
        auto pure = [&](R d[3], R &xx, R &yy, R &zz, R &ko) __attribute__((always_inline)) {
            if constexpr (LOP)
                ft.pure_lopsided(F, beta, d, xx, yy, zz, ko, lop);
            else
                ft.pure(F, d, xx, yy, zz, ko);
        };
        auto derivs1 = [&](R d[3], R &ko) __attribute__((always_inline)) {
            R xx, yy, zz;
            pure(d, xx, yy, zz, ko);
        };
        auto derivs2 = [&](R d[3], R dd[6], R &ko) __attribute__((always_inline)) {
            pure(d, dd[0], dd[3], dd[5], ko);
            ft.mixed(F, dd);
        };
        auto adv = [&](const R d[3]) __attribute__((always_inline)) {
            if constexpr (LOP)
                return beta[0] * lop[0] + beta[1] * lop[1] + beta[2] * lop[2];
            else
                return beta[0] * d[0] + beta[1] * d[1] + beta[2] * d[2];
        };
        // Monitor: constraint q at this point (0 where inactive) to a.cons,
        // and its |c|, c^2 summed over the wave (butterfly) into mred.
        // Called by every lane of the workgroup.
        double *cb = MON && a.cons ? a.cons + B.coffset : nullptr;
        R Mc[3] = {R(0), R(0), R(0)};   // M_i accumulated over the stages
        auto mon = [&](auto QC, R c_r) __attribute__((always_inline)) {
            constexpr int q = decltype(QC)::value;
            const double c = active ? double(c_r) : 0.0;
            if (active && cb)
                at(cb + q * fs, upt8) = c;
            double v1 = fabs(c), v2 = c * c;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                v1 += __shfl_xor(v1, off, 64);
                v2 += __shfl_xor(v2, off, 64);
            }
            if ((t & 63) == 0) {
                mred[(t >> 6) * 16 + 2 * q] = v1;
                mred[(t >> 6) * 16 + 2 * q + 1] = v2;
            }
        };

        // ---- shift: d beta (kept for the Lie-derivative terms), d d beta -> Gt
        R rG[3] = {R(0), R(0), R(0)};
        R divb = R(0);
        sfor<3>([&](auto K_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(K_c)::value;
            stage(std::integral_constant<int, BETAX + kk>{});
            New nw;
            if (active) {
                const Old o = old(BETAX + kk);
                const R Gam = R(at(ub + (GAMX + kk) * fs, upt8));
                R d[3], dd[6], ko;
                derivs2(d, dd, ko);
                sfor<3>([&](auto J_c) __attribute__((always_inline)) {
                    constexpr int jj = decltype(J_c)::value;
                    put(18 + 3 * kk + jj, d[jj]);
                });
                divb += d[kk];
                rG[kk] += symtrace(gi, dd);
                sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                    constexpr int ii = decltype(I_c)::value;
                    rG[ii] += R(1.0 / 3.0) * (gi[S(ii, 0)] * dd[S(0, kk)] + gi[S(ii, 1)] * dd[S(1, kk)]
                                              + gi[S(ii, 2)] * dd[S(2, kk)]);
                });
                const R kb = (a.advect_gauge ? adv(d) : R(0)) + ko
                           + (a.shift == Z4C_SHIFT_GAMMADRIVER ? Gam : R(0)) - R(a.eta) * beta[kk];
                nw = combine(kb, staged(), o);
            }
            ft.arrive();
            if (active)
                write(BETAX + kk, nw);
        });

        // ---- conformal metric
        R dg[3][6];
        R Rij[6];
        double vg[6];   // new conformal metric (stage), held for the det enforcement
        sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            constexpr int ii = SI(q), jj = SJ(q);
            stage(std::integral_constant<int, GXX + q>{});
            New nw;
            if (active) {
                const Old o = old(GXX + q);
                const R Aq = R(at(ub + (AXX + q) * fs, upt8));
                R d[3], dd[6], ko;
                derivs2(d, dd, ko);
                sfor<3>([&](auto K_c) __attribute__((always_inline)) {
                    constexpr int kk = decltype(K_c)::value;
                    dg[kk][q] = d[kk];
                });
                Rij[q] = R(-0.5) * symtrace(gi, dd);
                R lie = R(0);
                sfor<3>([&](auto K_c) __attribute__((always_inline)) {
                    constexpr int kk = decltype(K_c)::value;
                    lie += g[S(ii, kk)] * DB(kk, jj) + g[S(jj, kk)] * DB(kk, ii);
                });
                const R kg = adv(d) + ko - R(2) * alpha * Aq + lie
                           - R(2.0 / 3.0) * g[q] * divb;
                nw = combine(kg, staged(), o);
            }
            ft.arrive();
            if (active) {
                if constexpr (RK) {
                    vg[q] = nw.w;
                    write1(GXX + q, nw);
                } else {
                    write(GXX + q, nw);
                }
            }
        });
        if constexpr (RK) {
            if (active) {
                // det(gt) = 1
                const double det = vg[0] * (vg[3] * vg[5] - vg[4] * vg[4])
                                 - vg[1] * (vg[1] * vg[5] - vg[4] * vg[2])
                                 + vg[2] * (vg[1] * vg[4] - vg[3] * vg[2]);
                const double f = 1.0 / cbrt(det);
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    vg[q] *= f;
                    at(ob + (GXX + q) * fs, upt8) = vg[q];
                });
            }
        }

        // Christoffel symbols and the first-derivative part of the Ricci tensor.
        R Gd[3];
        if (active) {
            R Gl[3][6];
            sfor<3>([&](auto K_c) __attribute__((always_inline)) {
                constexpr int kk = decltype(K_c)::value;
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    constexpr int ii = SI(q), jj = SJ(q);
                    Gl[kk][q] = R(0.5) * (dg[ii][S(jj, kk)] + dg[jj][S(ii, kk)] - dg[kk][q]);
                });
            });
            R Gu[3][6];
            sfor<3>([&](auto K_c) __attribute__((always_inline)) {
                constexpr int kk = decltype(K_c)::value;
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    Gu[kk][q] = gi[S(kk, 0)] * Gl[0][q] + gi[S(kk, 1)] * Gl[1][q]
                              + gi[S(kk, 2)] * Gl[2][q];
                    put(6 * kk + q, Gu[kk][q]);
                });
                Gd[kk] = symtrace(gi, Gu[kk]);
            });
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                constexpr int ii = SI(q), jj = SJ(q);
                R s = R(0);
                sfor<3>([&](auto K_c) __attribute__((always_inline)) {
                    constexpr int kk = decltype(K_c)::value;
                    s += R(0.5) * Gd[kk] * (Gl[ii][S(jj, kk)] + Gl[jj][S(ii, kk)]);
                });
                Rij[q] += s;
            });
            // + sum_kl (Gu^k_{li} T_{jk}^l + Gu^k_{lj} T_{ik}^l + Gu^k_{il} T_{kj}^l),
            //   T_{ab}^c = gt^{cm} Gt_{a bm}
            sfor<3>([&](auto P0_c) __attribute__((always_inline)) {
                constexpr int p0 = decltype(P0_c)::value;
                sfor<3>([&](auto P1_c) __attribute__((always_inline)) {
                    constexpr int p1 = decltype(P1_c)::value;
                    R Tc[3];
                    sfor<3>([&](auto P2_c) __attribute__((always_inline)) {
                        constexpr int p2 = decltype(P2_c)::value;
                        Tc[p2] = gi[S(p2, 0)] * Gl[p0][S(p1, 0)] + gi[S(p2, 1)] * Gl[p0][S(p1, 1)]
                               + gi[S(p2, 2)] * Gl[p0][S(p1, 2)];
                    });
                    sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                        constexpr int q = decltype(Q_c)::value;
                        constexpr int ii = SI(q), jj = SJ(q);
                        R s = R(0);
                        sfor<3>([&](auto L_c) __attribute__((always_inline)) {
                            constexpr int l = decltype(L_c)::value;
                            if constexpr (jj == p0)
                                s += Gu[p1][S(l, ii)] * Tc[l];
                            if constexpr (ii == p0)
                                s += Gu[p1][S(l, jj)] * Tc[l];
                            if constexpr (jj == p1)
                                s += Gu[p0][S(ii, l)] * Tc[l];
                        });
                        Rij[q] += s;
                    });
                });
            });
            // Lie-derivative terms of Gamma-tilde
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                rG[ii] += -(Gd[0] * DB(ii, 0) + Gd[1] * DB(ii, 1) + Gd[2] * DB(ii, 2))
                        + R(2.0 / 3.0) * Gd[ii] * divb;
            });
        }

        const R kap1 = R(a.kappa1), kap2 = R(a.kappa2);
        // ---- Gamma-tilde: d_j Gt^k -> Ricci; damping
        sfor<3>([&](auto K_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(K_c)::value;
            stage(std::integral_constant<int, GAMX + kk>{});
            R Zk = R(0);
            if (active) {
                R d[3], ko;
                derivs1(d, ko);
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    constexpr int ii = SI(q), jj = SJ(q);
                    Rij[q] += R(0.5) * (g[S(kk, ii)] * d[jj] + g[S(kk, jj)] * d[ii]);
                });
                const R Gam = R(staged());
                rG[kk] += adv(d) + ko
                        - R(2) * alpha * kap1 * (Gam - Gd[kk]);
                if constexpr (MON)
                    Zk = R(0.5) * (Gam - Gd[kk]);
            }
            if constexpr (MON)
                mon(std::integral_constant<int, C_ZX + kk>{}, Zk);
        });

        // ---- lapse: alpha is complete; d_i d_j alpha - Gt^k_ij d_k alpha is
        // kept for the chi stage
        R dal[3], DDa[6];
        R Khat = R(0);
        stage(std::integral_constant<int, ALPHA>{});
        New nal;
        if (active) {
            const Old o = old(ALPHA);
            Khat = R(at(ub + KHAT * fs, upt8));
            R ko;
            derivs2(dal, DDa, ko);
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                DDa[q] -= GU(0, q) * dal[0] + GU(1, q) * dal[1] + GU(2, q) * dal[2];
            });
            R muL = R(0);
            if (a.lapse == Z4C_LAPSE_1PLUSLOG)
                muL = R(2) * alpha;
            else if (a.lapse == Z4C_LAPSE_HARMONIC)
                muL = alpha * alpha;
            const R ka = (a.advect_gauge ? adv(dal) : R(0)) + ko
                       - muL * Khat;
            nal = combine(ka, staged(), o);
            if constexpr (RK)
                nal.w = nal.w > a.alpha_floor ? nal.w : a.alpha_floor;
        }
        ft.arrive();
        if (active)
            write(ALPHA, nal);

        // ---- chi: R^chi_ij, D_i D_j alpha; chi is complete, and with it the
        // sources of Khat, Theta and At
        R Kpart = R(0), Tpart = R(0), Theta = R(0);
        R Hc = R(0);                  // monitor: Hamiltonian constraint
        stage(std::integral_constant<int, CHI>{});
        if (active) {
            const Old o = old(CHI);
            Theta = R(at(ub + THETA * fs, upt8));
            R A[6];
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                A[q] = R(at(ub + (AXX + q) * fs, upt8));
            });
            const R chi = R(staged());
            const R chis = chi > R(a.chi_floor) ? chi : R(a.chi_floor);
            const R ichi2 = R(0.5) / chis;          // 1 / (2 chi)
            const R K = Khat + R(2) * Theta;
            R dchi[3], dd[6], ko;
            derivs2(dchi, dd, ko);
            const R kc = adv(dchi) + ko
                       + R(2.0 / 3.0) * chi * (alpha * K - divb);
            New nchi = combine(kc, staged(), o);
            if constexpr (RK)
                nchi.w = nchi.w > a.chi_floor ? nchi.w : a.chi_floor;
            write(CHI, nchi);   // here: held to the end of this stage they spill
            {
                R dchi2 = R(0), ca = R(0);   // gt^{kl} d_k chi d_l (chi, alpha)
                sfor<3>([&](auto P0_c) __attribute__((always_inline)) {
                    constexpr int p0 = decltype(P0_c)::value;
                    const R v = gi[S(p0, 0)] * dchi[0] + gi[S(p0, 1)] * dchi[1]
                              + gi[S(p0, 2)] * dchi[2];
                    dchi2 += v * dchi[p0];
                    ca += v * dal[p0];
                });
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    dd[q] -= GU(0, q) * dchi[0] + GU(1, q) * dchi[1] + GU(2, q) * dchi[2];
                });
                const R trDD = symtrace(gi, dd);
                const R i4c2 = ichi2 * ichi2;   // 1 / (4 chi^2)
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    constexpr int ii = SI(q), jj = SJ(q);
                    Rij[q] += (dd[q] + g[q] * trDD) * ichi2
                            - (dchi[ii] * dchi[jj] + R(3) * g[q] * dchi2) * i4c2;
                    DDa[q] += (dchi[ii] * dal[jj] + dchi[jj] * dal[ii] - g[q] * ca) * ichi2;
                });
            }
            // matter
            R rho = R(0), Si[3] = {R(0), R(0), R(0)}, Sij[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
            if (a.matter) {
                const double *mb = a.matter + B.moffset;
                rho = R(at(mb, upt8));
                sfor<3>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    Si[q] = R(at(mb + (1 + q) * fs, upt8));
                });
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    Sij[q] = R(at(mb + (4 + q) * fs, upt8));
                });
            }
            const R trS = chi * symtrace(gi, Sij);
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                rG[ii] += R(-16) * pi * alpha
                        * (gi[S(ii, 0)] * Si[0] + gi[S(ii, 1)] * Si[1] + gi[S(ii, 2)] * Si[2]);
            });
            const R Rs = chi * symtrace(gi, Rij);
            Kpart = alpha * (K * K * R(1.0 / 3.0)) + R(4) * pi * alpha * (trS + rho)
                  + alpha * kap1 * (R(1) - kap2) * Theta - chi * symtrace(gi, DDa);
            Tpart = R(0.5) * alpha * (Rs + R(2.0 / 3.0) * K * K)
                  - alpha * (R(8) * pi * rho + kap1 * (R(2) + kap2) * Theta);
            if constexpr (MON)
                Hc = Rs + R(2.0 / 3.0) * K * K - R(16) * pi * rho;
            // chi [alpha (R - 8 pi S) - D D alpha]^tf
            R Y[6];
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                Y[q] = alpha * (Rij[q] - R(8) * pi * Sij[q]) - DDa[q];
            });
            const R trY = symtrace(gi, Y);
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                Y[q] = chi * (Y[q] - g[q] * trY * R(1.0 / 3.0));
            });
            // At^i_j, At^{ij}, At.At
            R Amix[3][3];
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                sfor<3>([&](auto J_c) __attribute__((always_inline)) {
                    constexpr int jj = decltype(J_c)::value;
                    Amix[ii][jj] = gi[S(ii, 0)] * A[S(0, jj)] + gi[S(ii, 1)] * A[S(1, jj)]
                                 + gi[S(ii, 2)] * A[S(2, jj)];
                });
            });
            // Gamma-tilde: 2 alpha Gt^i_jk At^jk - At^ij w_j with
            // w = 3 alpha / chi d chi + 2 d alpha
            R AA = R(0), w[3], gA[3] = {R(0), R(0), R(0)};
            const R c3 = R(6) * alpha * ichi2;
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                w[ii] = c3 * dchi[ii] + R(2) * dal[ii];
            });
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                constexpr int ii = SI(q), jj = SJ(q);
                const R up = Amix[ii][0] * gi[S(0, jj)] + Amix[ii][1] * gi[S(1, jj)]
                           + Amix[ii][2] * gi[S(2, jj)];
                const R up2 = R(SW(q)) * up;
                AA += A[q] * up2;
                gA[0] += GU(0, q) * up2;
                gA[1] += GU(1, q) * up2;
                gA[2] += GU(2, q) * up2;
                rG[ii] -= up * w[jj];
                if constexpr (ii != jj)
                    rG[jj] -= up * w[ii];
            });
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                rG[ii] += R(2) * alpha * gA[ii];
            });
            Kpart += alpha * AA;
            Tpart -= R(0.5) * alpha * AA;
            if constexpr (MON) {
                Hc -= AA;
                // M_i: -Gt_d^l At_li - Gt^l_ji At^j_l - 3/(2 chi) At^j_i d_j chi
                // - 8 pi S_i here; the At and K derivative terms in their stages
                sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                    constexpr int ii = decltype(I_c)::value;
                    R m = -(Gd[0] * A[S(0, ii)] + Gd[1] * A[S(1, ii)] + Gd[2] * A[S(2, ii)]);
                    sfor<3>([&](auto J_c) __attribute__((always_inline)) {
                        constexpr int jj = decltype(J_c)::value;
                        m -= GU(0, S(jj, ii)) * Amix[jj][0] + GU(1, S(jj, ii)) * Amix[jj][1]
                           + GU(2, S(jj, ii)) * Amix[jj][2];
                    });
                    m -= R(3) * ichi2 * (Amix[0][ii] * dchi[0] + Amix[1][ii] * dchi[1]
                                         + Amix[2][ii] * dchi[2]);
                    Mc[ii] += m - R(8) * pi * Si[ii];
                });
            }
            // At: + alpha (K At - 2 At At) + Lie
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                constexpr int ii = SI(q), jj = SJ(q);
                const R AAm = A[S(ii, 0)] * Amix[0][jj] + A[S(ii, 1)] * Amix[1][jj]
                            + A[S(ii, 2)] * Amix[2][jj];
                R la = R(0);
                sfor<3>([&](auto K_c) __attribute__((always_inline)) {
                    constexpr int kk = decltype(K_c)::value;
                    la += A[S(ii, kk)] * DB(kk, jj) + A[S(jj, kk)] * DB(kk, ii);
                });
                Y[q] += alpha * (K * A[q] - R(2) * AAm) + la - R(2.0 / 3.0) * A[q] * divb;
            });
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                put(18 + q, Y[q]);
            });
        }
        if constexpr (MON) {
            mon(std::integral_constant<int, C_H>{}, Hc);
            mon(std::integral_constant<int, C_THETA>{}, Theta);
        }

        // ---- Khat, Theta (their Gamma-tilde source terms); both complete
        double gam0[3] = {0.0, 0.0, 0.0};   // state of Gamma-tilde, completed after Theta
        Old gamo[3];
        sfor<2>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            stage(std::integral_constant<int, q == 0 ? KHAT : THETA>{});
            New nw;
            if (active) {
                const Old o = old(q == 0 ? KHAT : THETA);
                if constexpr (q == 1 && RK) {
                    sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                        constexpr int ii = decltype(I_c)::value;
                        gam0[ii] = at(ub + (GAMX + ii) * fs, upt8);
                        gamo[ii] = old(GAMX + ii);
                    });
                }
                R d[3], ko;
                derivs1(d, ko);
                const R c = q == 0 ? R(-4.0 / 3.0) * alpha : R(-2.0 / 3.0) * alpha;
                sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                    constexpr int ii = decltype(I_c)::value;
                    rG[ii] += c * (gi[S(ii, 0)] * d[0] + gi[S(ii, 1)] * d[1] + gi[S(ii, 2)] * d[2]);
                });
                if constexpr (MON) {   // -2/3 d_i K, K = Khat + 2 Theta
                    sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                        constexpr int ii = decltype(I_c)::value;
                        Mc[ii] -= R(q == 0 ? 2.0 / 3.0 : 4.0 / 3.0) * d[ii];
                    });
                }
                const R kq = adv(d) + ko + (q == 0 ? Kpart : Tpart);
                nw = combine(kq, staged(), o);
            }
            ft.arrive();
            if (active)
                write(q == 0 ? KHAT : THETA, nw);
        });
        // Gamma-tilde is complete
        if (active) {
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                write(GAMX + ii, combine(rG[ii], gam0[ii], gamo[ii]));
            });
        }

        // ---- At_ij; then tr(At) = 0 with the new conformal metric
        double vA[6], vn[6];
        sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            stage(std::integral_constant<int, AXX + q>{});
            New nw;
            if (active) {
                const Old o = old(AXX + q);
                if constexpr (q == 5 && RK) {
                    // the new conformal metric, as stored by this thread
                    unsigned upr = upt8;
                    asm volatile("" : "+v"(upr));
                    sfor<6>([&](auto P_c) __attribute__((always_inline)) {
                        constexpr int p = decltype(P_c)::value;
                        vn[p] = at(ob + (GXX + p) * fs, upr);
                    });
                }
                R d[3], ko;
                derivs1(d, ko);
                if constexpr (MON) {   // gt^{jk} d_k At_ij, At_ij = At_ji
                    constexpr int ii = SI(q), jj = SJ(q);
                    Mc[ii] += gi[S(jj, 0)] * d[0] + gi[S(jj, 1)] * d[1] + gi[S(jj, 2)] * d[2];
                    if constexpr (ii != jj)
                        Mc[jj] += gi[S(ii, 0)] * d[0] + gi[S(ii, 1)] * d[1] + gi[S(ii, 2)] * d[2];
                }
                const R kA = adv(d) + ko + get(18 + q);
                nw = combine(kA, staged(), o);
            }
            ft.arrive();
            if (active) {
                if constexpr (RK) {
                    vA[q] = nw.w;
                    write1(AXX + q, nw);
                } else {
                    write(AXX + q, nw);
                }
            }
        });
        if constexpr (RK) {
            if (active) {
                const double det = vn[0] * (vn[3] * vn[5] - vn[4] * vn[4])
                                 - vn[1] * (vn[1] * vn[5] - vn[4] * vn[2])
                                 + vn[2] * (vn[1] * vn[4] - vn[3] * vn[2]);
                const double id = 1.0 / det;
                const double gn[6] = {(vn[3] * vn[5] - vn[4] * vn[4]) * id,
                                      (vn[2] * vn[4] - vn[1] * vn[5]) * id,
                                      (vn[1] * vn[4] - vn[2] * vn[3]) * id,
                                      (vn[0] * vn[5] - vn[2] * vn[2]) * id,
                                      (vn[2] * vn[1] - vn[0] * vn[4]) * id,
                                      (vn[0] * vn[3] - vn[1] * vn[1]) * id};
                const double tr = gn[0] * vA[0] + gn[3] * vA[3] + gn[5] * vA[5]
                                + 2.0 * (gn[1] * vA[1] + gn[2] * vA[2] + gn[4] * vA[4]);
                sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                    constexpr int q = decltype(Q_c)::value;
                    at(ob + (AXX + q) * fs, upt8) = vA[q] - vn[q] * tr * (1.0 / 3.0);
                });
            }
        }
        if constexpr (MON) {
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                mon(std::integral_constant<int, C_MX + ii>{}, Mc[ii]);
            });
            __syncthreads();
            // per-tile sums, the waves in order (as the constraint kernel)
            if (t < 16) {
                double sum = 0.0;
                for (int w = 0; w < NT / 64; ++w)
                    sum += mred[w * 16 + t];
                a.partial[tile * 16LL + t] = sum;
            }
        }
    }
}

}  // namespace tile

// MODE_RHS or MODE_RK; WPE: waves per SIMD the kernel is compiled for.
template <int P, int WPE, typename R, int MODE, bool MON = false, bool LOP = false,
          bool NAIVE = false>
hipError_t launch_kernel(const StageArgs &a, hipStream_t s)
{
    constexpr int X = TILE_X, Y = TILE_Y, Z = TILE_Z;
    if (general_halo(a))
        tile::stage_kernel<P, X, Y, Z, WPE, R, MODE, true, MON, LOP, NAIVE>
            <<<a.ntiles, X * Y * Z, 0, s>>>(a);
    else
        tile::stage_kernel<P, X, Y, Z, WPE, R, MODE, false, MON, LOP, NAIVE>
            <<<a.ntiles, X * Y * Z, 0, s>>>(a);
    return hipGetLastError();
}

template <int P, int WPE, typename R, bool LOP = false>
hipError_t launch_variant(int mode, const StageArgs &a, hipStream_t s)
{
    return mode == MODE_RHS ? launch_kernel<P, WPE, R, MODE_RHS, false, LOP>(a, s)
                            : launch_kernel<P, WPE, R, MODE_RK, false, LOP>(a, s);
}

}  // namespace z4c
