// z4c_cons.h -- the constraint kernel (Sec. 4.1 monitoring; included by the
// per-variant translation units z4c_variants_*.hip).
#pragma once
#include "z4c_tile.h"

namespace z4c {
namespace tile {

// Sums of N values over a wave: lanes l with l mod (64 / N) = 0 end with that of
// value l / (64 / N).  A butterfly in which each half of the lanes goes on with
// half of the values, while there are several: N - 1 + log2(64 / N) exchanges
// instead of 6 N, and the same sums (N = 16: 96 x 24^3 blocks 304 -> 282 us).
template <int N>
__device__ __forceinline__ double wave_sums(double (&v)[N], unsigned lane)
{
    int off = 32;
#pragma unroll
    for (int n = N / 2; n >= 1; n >>= 1, off >>= 1) {
        const bool hi = lane & off;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const double keep = hi ? v[i + n] : v[i], give = hi ? v[i] : v[i + n];
            v[i] = keep + __shfl_xor(give, off, 64);
        }
    }
#pragma unroll
    for (; off >= 1; off >>= 1)
        v[0] += __shfl_xor(v[0], off, 64);
    return v[0];
}

// H, M_i, Theta and Z^i of the state at every interior point, and their
// per-tile sums of |c| and c^2.  chi is staged before the conformal metric
// and its derivatives wait in registers, so that the Christoffel symbols are
// needed in one place only (Ricci tensor, chi part, At contractions) and
// nothing is parked in LDS; then Gamma-tilde, Khat, Theta and At add their
// first derivatives.  What bounds it, as the stage kernel: latency.
// Measured (96 blocks of 24^3 with matter): 0.812 ms with the whole halo box
// in LDS, 400 registers and 8x8x8 tiles, 0.473 ms on 8x8x4 tiles, 0.327 ms
// in this form at two waves per SIMD (three, 168 registers and 53 spilled,
// 0.379 ms), 0.282 with the sums above, 0.269 without the points that only
// the dissipation reads.
template <int P, int TX, int TY, int TZ, int WPE, bool GEN>
__global__ void __launch_bounds__(TX *TY *TZ) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
cons_kernel(const StageArgs a)
{
    using D = ColDims<P, TX, TY, TZ>;
    using MZ = MixDimsZ<P, TX, TY, TZ>;
    using R = double;
    constexpr int NT = D::NT;
    __shared__ double pl[D::NPL];
    __shared__ double zc[D::NZC];
    __shared__ double zs[MZ::NZS];
    __shared__ double ys[MZ::NYS];
    __shared__ double red[(NT / 64) * 16];

    const int tile = my_tile();
    const unsigned t = threadIdx.x;
    const Tile T = table_entry(a.tiles, tile);
    const z4c_block B = table_entry(a.blocks, T.block);
    const int ng = B.ng;
    const int sy = B.nx + 2 * ng;
    const int sz = sy * (B.ny + 2 * ng);
    const int i = T.i0 + (int)(t % TX), j = T.j0 + (int)((t / TX) % TY), k = T.k0 + (int)(t / (TX * TY));
    const bool active = i < B.nx && j < B.ny && k < B.nz;
    const unsigned upt8 = 8u * (unsigned)((k + ng) * sz + (j + ng) * sy + (i + ng));
    const double *ub = a.u + B.offset;
    const long long fs = B.field_stride;
    const Fac<R> F = table_entry((const Fac<R> *)a.fac64, T.block);

    FieldTile<P, TX, TY, TZ, GEN, false> ft;   // no dissipation
    ft.setup(a, T, B, t, pl, zc, zs, ys);
    auto stage = [&](auto FC) __attribute__((always_inline)) {
        constexpr int FF = decltype(FC)::value;
        ft.template stage<FF, next_field<MODE_CONS>(FF)>();
    };
    auto derivs1 = [&](R d[3]) __attribute__((always_inline)) {
        R xx, yy, zz, ko;
        ft.pure(F, d, xx, yy, zz, ko);
    };
    auto derivs2 = [&](R d[3], R dd[6]) __attribute__((always_inline)) {
        R ko;
        ft.pure(F, d, dd[0], dd[3], dd[5], ko);
        ft.mixed(F, dd);
    };
    ft.st.template prefetch<mixed_field(CHI)>(CHI);

    // Conformal metric and its inverse.
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
    R cons[NCONS];
    sfor<NCONS>([&](auto Q_c) __attribute__((always_inline)) {
        cons[decltype(Q_c)::value] = R(0);
    });

    // ---- chi
    R chi = R(1), dchi[3], ddc[6];
    stage(std::integral_constant<int, CHI>{});
    if (active) {
        chi = ft.centre();
        derivs2(dchi, ddc);
    }

    // ---- conformal metric: d gt, d d gt -> Rt_ij (second-derivative part)
    R dg[3][6];
    R Rij[6];
    sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
        constexpr int q = decltype(Q_c)::value;
        stage(std::integral_constant<int, GXX + q>{});
        if (active) {
            R d[3], dd[6];
            derivs2(d, dd);
            sfor<3>([&](auto K_c) __attribute__((always_inline)) {
                constexpr int kk = decltype(K_c)::value;
                dg[kk][q] = d[kk];
            });
            Rij[q] = R(-0.5) * symtrace(gi, dd);
        }
    });

    // ---- Christoffel symbols Gl[k][ij] = Gt_{k ij}, Gu[k][ij] = Gt^k_{ij} and
    // everything they enter
    R Gd[3];
    R Rs = R(0), AA = R(0), rho = R(0);
    if (active) {
        R Gl[3][6], Gu[3][6];
        sfor<3>([&](auto K_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(K_c)::value;
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                constexpr int ii = SI(q), jj = SJ(q);
                Gl[kk][q] = R(0.5) * (dg[ii][S(jj, kk)] + dg[jj][S(ii, kk)] - dg[kk][q]);
            });
        });
        sfor<3>([&](auto K_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(K_c)::value;
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                Gu[kk][q] = gi[S(kk, 0)] * Gl[0][q] + gi[S(kk, 1)] * Gl[1][q]
                          + gi[S(kk, 2)] * Gl[2][q];
            });
            Gd[kk] = symtrace(gi, Gu[kk]);
        });
        // Rt_ij += 1/2 Gd^k (Gt_{ijk} + Gt_{jik})
        //        + sum_kl (Gu^k_{li} T_{jk}^l + Gu^k_{lj} T_{ik}^l + Gu^k_{il} T_{kj}^l),
        // T_{ab}^c = gt^{cm} Gt_{a bm}
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
        // R^chi_ij
        const R chis = chi > a.chi_floor ? chi : a.chi_floor;
        const R ichi2 = R(0.5) / chis, i4c2 = ichi2 * ichi2;   // 1 / (2 chi), 1 / (4 chi^2)
        R dchi2 = R(0);
        sfor<3>([&](auto P0_c) __attribute__((always_inline)) {
            constexpr int p0 = decltype(P0_c)::value;
            dchi2 += dchi[p0] * (gi[S(p0, 0)] * dchi[0] + gi[S(p0, 1)] * dchi[1]
                                 + gi[S(p0, 2)] * dchi[2]);
        });
        sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            ddc[q] -= Gu[0][q] * dchi[0] + Gu[1][q] * dchi[1] + Gu[2][q] * dchi[2];
        });
        const R trDD = symtrace(gi, ddc);
        sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            Rij[q] += (ddc[q] + g[q] * trDD) * ichi2
                    - (dchi[SI(q)] * dchi[SJ(q)] + R(3) * g[q] * dchi2) * i4c2;
        });
        Rs = chi * symtrace(gi, Rij);
        // At.At; M_i: -Gt_d^l At_li - Gt^l_ji At^j_l - 3/(2 chi) At^j_i d_j chi
        // - 8 pi S_i (At^j_l = gt^{jk} At_kl)
        R A[6], Amix[3][3];
        sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            A[q] = R(at(ub + (AXX + q) * fs, upt8));
        });
        sfor<3>([&](auto I_c) __attribute__((always_inline)) {
            constexpr int ii = decltype(I_c)::value;
            sfor<3>([&](auto J_c) __attribute__((always_inline)) {
                constexpr int jj = decltype(J_c)::value;
                Amix[ii][jj] = gi[S(ii, 0)] * A[S(0, jj)] + gi[S(ii, 1)] * A[S(1, jj)]
                             + gi[S(ii, 2)] * A[S(2, jj)];
            });
        });
        sfor<3>([&](auto I_c) __attribute__((always_inline)) {
            constexpr int ii = decltype(I_c)::value;
            sfor<3>([&](auto J_c) __attribute__((always_inline)) {
                constexpr int jj = decltype(J_c)::value;
                AA += Amix[ii][jj] * Amix[jj][ii];
            });
        });
        R Si[3] = {R(0), R(0), R(0)};
        if (a.matter) {
            const double *mb = a.matter + B.moffset;
            rho = R(at(mb, upt8));
            sfor<3>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                Si[q] = R(at(mb + (1 + q) * fs, upt8));
            });
        }
        sfor<3>([&](auto I_c) __attribute__((always_inline)) {
            constexpr int ii = decltype(I_c)::value;
            R m = -(Gd[0] * A[S(0, ii)] + Gd[1] * A[S(1, ii)] + Gd[2] * A[S(2, ii)]);
            sfor<3>([&](auto J_c) __attribute__((always_inline)) {
                constexpr int jj = decltype(J_c)::value;
                m -= Gu[0][S(jj, ii)] * Amix[jj][0] + Gu[1][S(jj, ii)] * Amix[jj][1]
                   + Gu[2][S(jj, ii)] * Amix[jj][2];
            });
            m -= R(3) * ichi2 * (Amix[0][ii] * dchi[0] + Amix[1][ii] * dchi[1]
                                 + Amix[2][ii] * dchi[2]);
            cons[C_MX + ii] = m - R(8) * R(PI) * Si[ii];
        });
    }

    // ---- Gamma-tilde: chi gt^{ij} gt_ki d_j Gt^k = chi d_k Gt^k of the Ricci
    // scalar; Z^i
    sfor<3>([&](auto K_c) __attribute__((always_inline)) {
        constexpr int kk = decltype(K_c)::value;
        stage(std::integral_constant<int, GAMX + kk>{});
        if (active) {
            R d[3];
            derivs1(d);
            R s = R(0);   // gt^{ij} 1/2 (gt_ki d_j + gt_kj d_i) Gt^k
            sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
                constexpr int q = decltype(Q_c)::value;
                constexpr int ii = SI(q), jj = SJ(q);
                s += R(SW(q)) * gi[q] * (R(0.5) * (g[S(kk, ii)] * d[jj] + g[S(kk, jj)] * d[ii]));
            });
            Rs += chi * s;
            cons[C_ZX + kk] = R(0.5) * (ft.centre() - Gd[kk]);
        }
    });

    // ---- Khat, Theta: -2/3 d_i K, K = Khat + 2 Theta
    R KT[2] = {R(0), R(0)};
    sfor<2>([&](auto Q_c) __attribute__((always_inline)) {
        constexpr int q = decltype(Q_c)::value;
        stage(std::integral_constant<int, q == 0 ? KHAT : THETA>{});
        if (active) {
            R d[3];
            derivs1(d);
            KT[q] = ft.centre();
            sfor<3>([&](auto I_c) __attribute__((always_inline)) {
                constexpr int ii = decltype(I_c)::value;
                cons[C_MX + ii] -= R(q == 0 ? 2.0 / 3.0 : 4.0 / 3.0) * d[ii];
            });
        }
    });
    if (active) {
        const R K = KT[0] + R(2) * KT[1];
        cons[C_H] = Rs + R(2.0 / 3.0) * K * K - AA - R(16) * R(PI) * rho;
        cons[C_THETA] = KT[1];
    }

    // ---- At_ij: gt^{jk} d_k At_ij
    sfor<6>([&](auto Q_c) __attribute__((always_inline)) {
        constexpr int q = decltype(Q_c)::value;
        stage(std::integral_constant<int, AXX + q>{});
        if (active) {
            R d[3];
            derivs1(d);
            constexpr int ii = SI(q), jj = SJ(q);
            cons[C_MX + ii] += gi[S(jj, 0)] * d[0] + gi[S(jj, 1)] * d[1] + gi[S(jj, 2)] * d[2];
            if constexpr (ii != jj)
                cons[C_MX + jj] += gi[S(ii, 0)] * d[0] + gi[S(ii, 1)] * d[1] + gi[S(ii, 2)] * d[2];
        }
    });

    // ---- output
    if (active && a.out) {
        double *cb = a.out + B.coffset;
        sfor<NCONS>([&](auto Q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(Q_c)::value;
            at(cb + q * fs, upt8) = cons[q];
        });
    }
    // Per-tile sums of |c| and c^2 in a fixed order: over the wave, then the
    // waves in order.
    double v[16];
    sfor<NCONS>([&](auto Q_c) __attribute__((always_inline)) {
        constexpr int q = decltype(Q_c)::value;
        v[2 * q] = fabs(cons[q]);
        v[2 * q + 1] = cons[q] * cons[q];
    });
    const double sum = wave_sums<16>(v, t & 63);
    if ((t & 3) == 0)
        red[t >> 2] = sum;   // value (t & 63) >> 2 of wave t >> 6
    __syncthreads();
    if (t < 16) {
        double s = 0.0;
        for (int w = 0; w < NT / 64; ++w)
            s += red[w * 16 + t];
        a.partial[tile * 16LL + t] = s;
    }
}

}  // namespace tile

template <int P, int WPE>
hipError_t launch_cons(const StageArgs &a, hipStream_t s)
{
    constexpr int X = TILE_X, Y = TILE_Y, Z = TILE_Z;
    if (general_halo(a))
        tile::cons_kernel<P, X, Y, Z, WPE, true><<<a.ntiles, X * Y * Z, 0, s>>>(a);
    else
        tile::cons_kernel<P, X, Y, Z, WPE, false><<<a.ntiles, X * Y * Z, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace z4c
