// Star-shaped contours (builder-defined extension: one radius per table direction)
//
// One wave per contour. The table directions stay fixed in space (no rotation). Per iteration the
// Philox pair draws pick directions k; each pair's rays run along +T_k with radius R_k and along
// -T_k with the radius of the antipodal direction, with the sphere's radial points
// s = (R + dR/2) ((l + xi)/L)^(1/d) (L = 16: one DPP row of lanes per ray pair). With the per-point
// weight q(R) = (2R)^-d omega_d (R + dR/2)^d / (M L): E = sum q S I, g_c = sum q (-dS/dr I u), and
// every sampled direction k collects g_k = sum over its rays of q (B_R,ray - (d/R_k) A_ray)
// (rays that drew the same direction are summed in ray order by the first of them, so the result
// does not depend on timing). Step: c -= (eps/2) g_c; R_k -= (eps/2) D g_k + min(1, eps lambda / 2)
// (R_k - mean of its graph neighbours), from the old radii (double-buffered in LDS).
#include "evolve_core.h"

namespace snk {

namespace {

template <int DIM>
__host__ __device__ __forceinline__ int star_lds_floats(int D, int M, int NT, bool few = false) {
    const int per = (draw_floats(NT, M / 2) + 3) & ~3;
    return per + 4 * D + 2 + 2 * M + (M / 2) * (2 + DIM) * (few ? 2 : 1) + 8 * (NT / 64);
}

// Rows of the neighbour table that a lane of the FEW kernel keeps.
constexpr int kStarRows = 6;

// NT threads per contour (64: one wave; 128: two waves, whose partial sums meet in LDS in wave
// order).
//
// FEW: no more contours than the chip holds with 256 registers per lane, D <= kStarRows NT, neighbour rows of one
// chunk, M / 2 <= NT. An iteration is a chain of waits there (two gathers, the rays' table entries, two reads of
// neighbour rows, LDS in between) with one or two waves per SIMD to cover them. So the registers take what shortens
// the chain: the neighbour rows stay in them for the whole launch, four pair-points' gathers are in flight instead
// of two, and the next iteration's table entries are read during this one. 600 contours, D 642, 60 iterations:
// 560 -> 514 us; what is left is 1,470 vector instructions per wave and iteration, on half of the SIMDs for two
// waves, and the chain through LDS. With more contours the other kernel holds four waves per SIMD.
template <int DIM, int LAYOUT, int NT, bool FEW>
__global__ __launch_bounds__(NT, FEW ? 2 : (NT == 128 ? 4 : 1)) void star_kernel(EvolveArgs a, StarArgs sa) {
    extern __shared__ float lds[];
    constexpr float RHO = DIM == 3 ? 0.79370052598409973738f : 0.70710678118654752440f;
    constexpr float BALL = DIM == 3 ? 4.18879020478639098462f : 3.14159265358979323846f;
    const JobParams &p = a.p;
    const int cid = blockIdx.x;
    if (cid >= a.n) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    constexpr int NW = NT / 64;
    const int D = p.D, M = p.M, MH = M / 2, L = p.L;
    DevContour *slot = a.st + cid;
    DevContour s = uniform_copy(slot);
    const int n0 = s.iters;
    const int budget = (s.status & 0x0f) == SNK_ACTIVE ? a.n_iter : 0;
    const int per = (draw_floats(NT, MH) + 3) & ~3;
    const Draws dr(lds, NT, MH);
    // two radius buffers of D + 1 entries: entry D stays +0, so a neighbour row's padding (index D)
    // reads a zero
    float *Ra = lds + per;
    float *Rb = Ra + D + 1;
    float *gk = Rb + D + 1;
    int *ray_dir = reinterpret_cast<int *>(gk + D);
    float *ray_g = reinterpret_cast<float *>(ray_dir + M);
    // this iteration's ray pairs: direction, antipode, unit vector
    int *rk = reinterpret_cast<int *>(ray_g + M);
    int *rka = rk + MH;
    float *ru = reinterpret_cast<float *>(rka + MH);
    const int pairs_words = MH * (2 + DIM);                       // FEW: of the second buffer's offset
    float *red = ru + MH * DIM + (FEW ? pairs_words : 0);         // per-wave partials, 8 per wave
    // lowest ray of each direction this iteration (INT_MAX for none; reset by that ray after use)
    int *own = reinterpret_cast<int *>(red + 8 * NW);
    float *Rg = sa.Rk + (long)cid * D;
    for (int k = t; k < D; k += NT) {
        Ra[k] = Rg[k];
        gk[k] = 0.0f;
        own[k] = 0x7fffffff;
    }
    if (t == 0) {
        Ra[D] = 0.0f;
        Rb[D] = 0.0f;
    }
    const Vol<DIM, LAYOUT> vol(p.g);
    const int nvol[3] = {p.g.nx, p.g.ny, p.g.nz};
    const float inv_h[3] = {p.g.inv_h[0], p.g.inv_h[1], p.g.inv_h[2]};
    const float hh[3] = {p.g.h[0], p.g.h[1], p.g.h[2]};
    const uint32_t id = s.id;
    if (budget > 0) draws_phase1<DIM, NT, false>(dr, 0, (uint32_t)(n0 + 1), id, p, t);
    __syncthreads();
    // largest radius (interior test) and the clamp flag of the radii
    float rmax = 0.0f;
    for (int k = t; k < D; k += NT) rmax = fmaxf(rmax, Ra[k]);
    rmax = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_max_to_63(rmax)), 63));
    if constexpr (NW > 1) {
        if (lane == 0) red[wave * 8] = rmax;
        __syncthreads();
        rmax = red[0];
        for (int w = 1; w < NW; ++w) rmax = fmaxf(rmax, red[w * 8]);
        __syncthreads();
    }

    int anc[3] = {s.anc[0], s.anc[1], s.anc[2]};
    float off[3] = {s.off[0], s.off[1], s.off[2]};
    float Rmean = s.R;
    int n = n0;
    uint8_t status = s.status;
    int streak = s.streak;
    float e_mc = s.e_mc;
    const float invL = 1.0f / (float)L;
    const float inv_ml = 1.0f / (float)(M * L);
    const float tol2 = p.conv_tol * p.conv_tol;
    const float hd = 0.5f * RHO * p.dR, hD = 0.5f * p.dR;
    int ran = 0;
    float *Rold = Ra, *Rnew = Rb;
    const uint4 *nbrow = reinterpret_cast<const uint4 *>(sa.nb);
    uint4 kept[FEW ? kStarRows : 1];
    if constexpr (FEW) {
#pragma unroll
        for (int b = 0; b < kStarRows; ++b) kept[b] = nbrow[min(t + NT * b, D - 1)];
        if (budget > 0 && t < MH) {
            const int k = __float_as_int(dr.pu[t].x);
            rk[t] = k;
            rka[t] = sa.anti[k];
#pragma unroll
            for (int ax = 0; ax < DIM; ++ax) ru[t * DIM + ax] = p.dirs[k * DIM + ax];
        }
    }

    for (int it = 0; it < budget && (status & 0x0f) == SNK_ACTIVE; ++it) {
        const int blk = it / dr.K, sl = it - blk * dr.K;
        if (sl == 0) draws_phase1<DIM, NT, false>(dr, (blk + 1) & 1, (uint32_t)(n0 + 1 + (blk + 1) * dr.K), id, p, t);
        const float4 *pu = dr.pu + dr.slot(blk & 1, sl) * MH;
        Frame<DIM> fr;
        long base = 0;
        const long stride[3] = {1, vol.nx, vol.nxy};
        bool interior = true;
        const float ext_r = rmax + 0.5f * p.dR;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            fr.anc[ax] = anc[ax];
            fr.off[ax] = off[ax];
        }
#pragma unroll
        for (int ax = 0; ax < DIM; ++ax) {
            base += (long)anc[ax] * stride[ax];
            const float ext = fmaf(ext_r * inv_h[ax], 1.0001f, 1e-3f);
            interior = interior && (off[ax] - ext > (float)(-anc[ax])) && (off[ax] + ext < (float)(nvol[ax] - 1 - anc[ax]));
        }
        fr.base = base;
        // the ray pairs' tables entries, once per iteration (the pair-points below read them from LDS)
        if constexpr (!FEW) {
            for (int m = t; m < MH; m += NT) {
                const int k = __float_as_int(pu[m].x);
                rk[m] = k;
                rka[m] = sa.anti[k];
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) ru[m * DIM + ax] = p.dirs[k * DIM + ax];
            }
        }
        __syncthreads();
        // FEW: the next iteration's entries, on their way until this one's pair-points are done (its draws are
        // there: of this block, or of the next, which the block's first iteration drew before the barrier)
        int next_k = 0, next_ka = 0;
        float next_u[3] = {0.0f, 0.0f, 0.0f};
        if constexpr (FEW) {
            if (t < MH) {
                const int sn = sl + 1 == dr.K ? dr.slot((blk + 1) & 1, 0) : dr.slot(blk & 1, sl + 1);
                next_k = __float_as_int(dr.pu[sn * MH + t].x);
                next_ka = sa.anti[next_k];
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) next_u[ax] = p.dirs[next_k * DIM + ax];
            }
        }
        float accE = 0.0f, accc[3] = {0.0f, 0.0f, 0.0f};
        // pair-points q = t + NT j: pair m = q / 16, radial index l = q % 16 (one DPP row per pair);
        // H of them in flight, consumed in order
        constexpr int H = FEW ? 4 : 2;
        const int PP = MH * L;
        for (int q0 = t; q0 - t < PP; q0 += H * NT) {
            Corners<DIM> cr[H][2];
            float fv[H][2][3], Rv[H][2], ev[H], uv[H][3];
            int mv2[H], lv[H], kv[H][2];
            bool on[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int q = q0 + NT * h;
                on[h] = q < PP;
                if (!on[h]) continue;
                const int m = q >> 4, l = q & 15;
                mv2[h] = m;
                lv[h] = l;
                const int at = FEW && (it & 1) ? pairs_words : 0;
                const int k = rk[at + m], ka = rka[at + m];
                kv[h][0] = k;
                kv[h][1] = ka;
                float du[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) uv[h][ax] = 0.0f;
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) {
                    uv[h][ax] = ru[at + m * DIM + ax];
                    du[ax] = uv[h][ax] * inv_h[ax];
                }
                const float e = cube_or_square_root<DIM>(((float)l + pu[m].w) * invL);
                ev[h] = e;
#pragma unroll
                for (int sg = 0; sg < 2; ++sg) {
                    const float R = Rold[sg ? ka : k];
                    const float smax = R + 0.5f * p.dR;
                    const float rad = smax * e;
                    float w[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int ax = 0; ax < DIM; ++ax) w[ax] = fmaf(sg ? -rad : rad, du[ax], off[ax]);
                    Rv[h][sg] = R;
                    if (interior)
                        vol.load(locate<DIM, false, Vol<DIM, LAYOUT>::kSmall>(fr, nvol, vol.nx, vol.nxy, w, fv[h][sg]),
                                 fr.base, cr[h][sg]);
                    else
                        vol.load(locate<DIM, true, Vol<DIM, LAYOUT>::kSmall>(fr, nvol, vol.nx, vol.nxy, w, fv[h][sg]),
                                 0, cr[h][sg]);
                }
            }
#pragma unroll
            for (int h = 0; h < H; ++h) {
                if (!on[h]) continue;
                const int m = mv2[h], l = lv[h];
                const float e = ev[h];
                float Ival[2], Sv[2], cCv[2], cRv[2], qv[2];
#pragma unroll
                for (int sg = 0; sg < 2; ++sg) {
                    const float R = Rv[h][sg];
                    const float smax = R + 0.5f * p.dR;
                    const float I = trilerp<DIM>(cr[h][sg], fv[h][sg]);
                    const float d1 = fmaf(smax, e, -RHO * R), d2 = fmaf(smax, e, -R);
                    const float is = p.in_slope, os = p.out_slope;
                    const bool r1 = d1 >= -hd && d1 < hd;
                    const bool r2 = d2 >= -hD && d2 < hD;
                    const float sin_ = __builtin_amdgcn_fmed3f(d1 * is, -1.0f, 1.0f);
                    const float sout = __builtin_amdgcn_fmed3f(fmaf(-d2, os, 0.5f), 0.0f, 1.0f);
                    const float inv2R = __builtin_amdgcn_rcpf(2.0f * R);
                    float nrm = inv2R, sm_d = smax;
#pragma unroll
                    for (int i = 1; i < DIM; ++i) {
                        nrm *= inv2R;
                        sm_d *= smax;
                    }
                    Ival[sg] = I;
                    Sv[sg] = fminf(sin_, sout);
                    cCv[sg] = r1 ? is : (r2 ? -os : 0.0f);
                    cRv[sg] = r1 ? -RHO * is : -cCv[sg];
                    qv[sg] = BALL * sm_d * nrm * inv_ml;
                }
#pragma unroll
                for (int sg = 0; sg < 2; ++sg) {
                    const float qI = qv[sg] * Ival[sg];
                    accE = fmaf(Sv[sg], qI, accE);
                    const float gcs = -cCv[sg] * qI * (sg ? -1.0f : 1.0f);
#pragma unroll
                    for (int ax = 0; ax < DIM; ++ax) accc[ax] = fmaf(gcs, uv[h][ax], accc[ax]);
                }
                // per-ray sums over the row's 16 radial points
                float Ap = row_sum16(Sv[0] * Ival[0]), Bp = row_sum16(cRv[0] * Ival[0]);
                float Am = row_sum16(Sv[1] * Ival[1]), Bm = row_sum16(cRv[1] * Ival[1]);
                if (l == 0) {
                    ray_dir[2 * m] = kv[h][0];
                    ray_g[2 * m] = qv[0] * (Bp - ((float)DIM / Rv[h][0]) * Ap);
                    ray_dir[2 * m + 1] = kv[h][1];
                    ray_g[2 * m + 1] = qv[1] * (Bm - ((float)DIM / Rv[h][1]) * Am);
                }
            }
        }
        if constexpr (FEW) {
            // into the buffer that the last iteration read
            const int to = (it + 1) & 1 ? pairs_words : 0;
            if (t < MH) {
                rk[to + t] = next_k;
                rka[to + t] = next_ka;
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) ru[to + t * DIM + ax] = next_u[ax];
            }
        }
        float E = 0.0f, gc[3] = {0.0f, 0.0f, 0.0f};
        if constexpr (NW == 1) {
            E = wave_sum(accE);
#pragma unroll
            for (int ax = 0; ax < DIM; ++ax) gc[ax] = wave_sum(accc[ax]);
        } else {
            const float wE = wave_sum_to_63(accE);
            float wc[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ax = 0; ax < DIM; ++ax) wc[ax] = wave_sum_to_63(accc[ax]);
            if (lane == 63) {
                red[wave * 8] = wE;
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) red[wave * 8 + 1 + ax] = wc[ax];
            }
            __syncthreads();
            E = red[0];
#pragma unroll
            for (int ax = 0; ax < DIM; ++ax) gc[ax] = red[1 + ax];
            for (int w = 1; w < NW; ++w) {
                E += red[w * 8];
#pragma unroll
                for (int ax = 0; ax < DIM; ++ax) gc[ax] += red[w * 8 + 1 + ax];
            }
        }
        __syncthreads();
        // sampled directions: the first ray of each direction sums its rays in order (the sum starts
        // at +0, so it is never -0 and adding +0 leaves it unchanged).
        if (M <= 64) {
            // all rays in wave 0: the lowest ray of each direction comes from an LDS minimum; the few
            // later rays of a direction are then added, lowest first, by that direction's first ray
            if (wave == 0) {
                const bool has = lane < M;
                const int dk = has ? ray_dir[lane] : 0;
                const float gr = has ? ray_g[lane] : 0.0f;
                if (has) atomicMin(&own[dk], lane);
                // one wave's LDS operations complete in order: every lane's minimum is in
                const bool first = has && own[dk] == lane;
                float g = 0.0f + gr;
                uint64_t later = __builtin_amdgcn_ballot_w64(has && !first);
                while (later) {
                    const int j = __builtin_amdgcn_readfirstlane(__builtin_ctzll(later));
                    later &= later - 1;
                    const int dj = __builtin_amdgcn_readlane(dk, j);
                    const float gj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gr), j));
                    if (first && dk == dj) g += gj;
                }
                if (first) {
                    gk[dk] = g;
                    own[dk] = 0x7fffffff;
                }
            }
        } else {
            // Every lane walks all rays, eight at a time with their loads issued together and no branch
            // on the loaded values (a ray of another direction adds +0)
            for (int r = t; r < M; r += NT) {
                const int dk = ray_dir[r];
                bool first = true;
                float g = 0.0f;
                int r2 = 0;
                for (; r2 + 8 <= M; r2 += 8) {
                    int dd[8];
                    float gg[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        dd[u] = ray_dir[r2 + u];
                        gg[u] = ray_g[r2 + u];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const bool same = dd[u] == dk;
                        first = first && !(same && r2 + u < r);
                        g += same && r2 + u >= r ? gg[u] : 0.0f;
                    }
                }
                for (; r2 < M; ++r2) {
                    const bool same = ray_dir[r2] == dk;
                    first = first && !(same && r2 < r);
                    g += same && r2 >= r ? ray_g[r2] : 0.0f;
                }
                if (first) gk[dk] = g;
            }
        }
        __syncthreads();
        n += 1;
        const float eps = p.eps0 * __builtin_amdgcn_rsqf((float)n);
        const float half_eps = 0.5f * eps;
        const float relax = fminf(1.0f, half_eps * sa.lambda);
        float mv = 0.0f, sum = 0.0f, mx = 0.0f;
        int clamped = 0, finite_r = 1;
        // neighbour rows of four directions are loaded before any of them is used; every entry is
        // read without a branch (the padding index D reads +0, which leaves the sum unchanged), so
        // a row's LDS reads are all issued before the first is added
        // (a direction past D loads the last row, unused)
        constexpr int ROWS = FEW ? kStarRows : 4;
        for (int k0 = t; k0 < D; k0 += ROWS * NT) {
            uint4 pre[ROWS];
#pragma unroll
            for (int b = 0; b < ROWS; ++b) pre[b] = FEW ? kept[b] : nbrow[min(k0 + NT * b, D - 1) * sa.nb_chunks];
#pragma unroll
            for (int b = 0; b < ROWS; ++b) {
                const int k = k0 + NT * b;
                if (k < D) {
                    // neighbour mean in the rows' order
                    float ms = 0.0f;
                    int cnt = 0;
                    for (int ch = 0; ch < (FEW ? 1 : sa.nb_chunks); ++ch) {
                        const uint4 w = ch == 0 ? pre[b] : nbrow[k * sa.nb_chunks + ch];
                        const uint32_t wv[4] = {w.x, w.y, w.z, w.w};
                        float rv[8];
#pragma unroll
                        for (int t8 = 0; t8 < 8; ++t8) {
                            const uint32_t j = (wv[t8 >> 1] >> (16 * (t8 & 1))) & 0xffffu;
                            rv[t8] = Rold[j];
                            cnt += j != (uint32_t)D;
                        }
#pragma unroll
                        for (int t8 = 0; t8 < 8; ++t8) ms += rv[t8];
                    }
                    const float Rk0 = Rold[k];
                    const float mk = cnt > 0 ? ms / (float)cnt : Rk0;
                    float Rn = Rk0 - half_eps * (float)D * gk[k] - relax * (Rk0 - mk);
                    if (Rn < p.r_lo) {
                        Rn = p.r_lo;
                        clamped = 1;
                    }
                    if (Rn > p.r_hi) {
                        Rn = p.r_hi;
                        clamped = 1;
                    }
                    finite_r = finite_r && isfinite(Rn);
                    mv = fmaxf(mv, fabsf(Rn - Rk0));
                    sum += Rn;
                    mx = fmaxf(mx, Rn);
                    Rnew[k] = Rn;
                    gk[k] = 0.0f;
                }
            }
        }
        mv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_max_to_63(mv)), 63));
        mx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_max_to_63(mx)), 63));
        clamped = __builtin_amdgcn_ballot_w64(clamped != 0) != 0;
        bool fin_r = __builtin_amdgcn_ballot_w64(!finite_r) == 0;
        if constexpr (NW == 1) {
            sum = wave_sum(sum);
        } else {
            const float ws = wave_sum_to_63(sum);
            if (lane == 63) {
                red[wave * 8] = mv;
                red[wave * 8 + 1] = mx;
                red[wave * 8 + 2] = ws;
                red[wave * 8 + 3] = clamped ? 1.0f : 0.0f;
                red[wave * 8 + 4] = fin_r ? 1.0f : 0.0f;
            }
            __syncthreads();
            mv = red[0];
            mx = red[1];
            sum = red[2];
            clamped = red[3] != 0.0f;
            fin_r = red[4] != 0.0f;
            for (int w = 1; w < NW; ++w) {
                mv = fmaxf(mv, red[w * 8]);
                mx = fmaxf(mx, red[w * 8 + 1]);
                sum += red[w * 8 + 2];
                clamped = clamped || red[w * 8 + 3] != 0.0f;
                fin_r = fin_r && red[w * 8 + 4] != 0.0f;
            }
        }
        rmax = mx;
        Rmean = sum / (float)D;
        e_mc = E;
        float dc2 = 0.0f;
        bool finite = fin_r && isfinite(E);
#pragma unroll
        for (int ax = 0; ax < DIM; ++ax) {
            const float dcp = -half_eps * gc[ax];
            dc2 = fmaf(dcp, dcp, dc2);
            off[ax] += dcp * inv_h[ax];
            finite = finite && isfinite(off[ax]);
        }
        uint8_t flag = (status & SNK_CLAMPED) | (clamped ? SNK_CLAMPED : 0);
        uint8_t st = SNK_ACTIVE;
        if (!finite) {
            st = SNK_NONFINITE;
        } else {
#pragma unroll
            for (int ax = 0; ax < DIM; ++ax) {
                if (fabsf(off[ax]) >= 0.5f) {
                    const float kk = rintf(off[ax]);
                    anc[ax] += (int)kk;
                    off[ax] -= kk;
                }
                if (off[ax] < (float)(-anc[ax]) || off[ax] > (float)(nvol[ax] - 1 - anc[ax])) st = SNK_OUT;
            }
        }
        if (st == SNK_ACTIVE) {
            const bool small = mv * mv < tol2 && dc2 < tol2;
            streak = small ? min(streak + 1, 255) : 0;
            if (p.conv_window > 0 && streak >= p.conv_window) st = SNK_CONVERGED;
        }
        status = (uint8_t)uni<64>((int)(st | flag));
        streak = uni<64>(streak);
#pragma unroll
        for (int ax = 0; ax < DIM; ++ax) {
            off[ax] = uni<64>(off[ax]);
            anc[ax] = uni<64>(anc[ax]);
        }
        float *t = Rold;
        Rold = Rnew;
        Rnew = t;
        ++ran;
        // no barrier here: the next iteration first writes the ray tables and the next block's
        // draws, which nothing reads after this iteration's last barrier, and its barrier after
        // the ray tables orders everything else
    }
    if (budget > 0) {
        for (int k = t; k < D; k += NT) Rg[k] = Rold[k];
        if (t == 0) {
            DevContour o = s;
            for (int i = 0; i < 3; ++i) {
                o.anc[i] = anc[i];
                o.off[i] = off[i];
            }
            o.R = Rmean;
            o.e_mc = e_mc;
            o.iters = n;
            o.status = status;
            o.streak = (uint8_t)streak;
            *slot = o;
            atomicAdd(a.counter, (unsigned long long)ran);
        }
    }
}

template <int DIM, int NT, bool FEW>
hipError_t launch_star_t(const EvolveArgs &a, const StarArgs &sa, int layout, hipStream_t s) {
    const size_t lds = sizeof(float) * (size_t)star_lds_floats<DIM>(a.p.D, a.p.M, NT, FEW);
    switch (layout) {
        case kBufferQuad:
            hipLaunchKernelGGL((star_kernel<DIM, kBufferQuad, NT, FEW>), dim3(a.n), dim3(NT), lds, s, a, sa);
            break;
        case kBufferPair:
            hipLaunchKernelGGL((star_kernel<DIM, kBufferPair, NT, FEW>), dim3(a.n), dim3(NT), lds, s, a, sa);
            break;
        case kBufferPlain:
            hipLaunchKernelGGL((star_kernel<DIM, kBufferPlain, NT, FEW>), dim3(a.n), dim3(NT), lds, s, a, sa);
            break;
        default:
            hipLaunchKernelGGL((star_kernel<DIM, kGlobalPlain, NT, FEW>), dim3(a.n), dim3(NT), lds, s, a, sa);
            break;
    }
    return hipGetLastError();
}

template <int DIM, int NT>
hipError_t launch_star_n(const EvolveArgs &a, const StarArgs &sa, int layout, int cus, hipStream_t s) {
    const bool few = (long)a.n * (NT / 64) <= 8l * cus && a.p.D <= kStarRows * NT && sa.nb_chunks == 1 &&
                     a.p.M / 2 <= NT && sizeof(float) * star_lds_floats<DIM>(a.p.D, a.p.M, NT, true) <= 65536;
    return few ? launch_star_t<DIM, NT, true>(a, sa, layout, s) : launch_star_t<DIM, NT, false>(a, sa, layout, s);
}

template <int DIM>
hipError_t launch_star_d(const EvolveArgs &a, const StarArgs &sa, int lanes, int layout, int cus, hipStream_t s) {
    if (lanes == 128) return launch_star_n<DIM, 128>(a, sa, layout, cus, s);
    if (lanes == 64) return launch_star_n<DIM, 64>(a, sa, layout, cus, s);
    return hipErrorInvalidValue;
}

}  // namespace

namespace {
__global__ __launch_bounds__(256) void star_init_kernel(const DevContour *st, float *Rk, int n, int D) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < (long)n * D) Rk[i] = st[i / D].R;
}
}  // namespace

hipError_t launch_star_init(const DevContour *st, float *Rk, int n, int D, hipStream_t s) {
    const long total = (long)n * D;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(star_init_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, st, Rk, n, D);
    return hipGetLastError();
}

hipError_t launch_star(const EvolveArgs &a, const StarArgs &sa, int dim, int lanes, int layout, int cus, hipStream_t s) {
    if (a.n <= 0 || a.n_iter <= 0) return hipSuccess;
    return dim == 2 ? launch_star_d<2>(a, sa, lanes, layout, cus, s) : launch_star_d<3>(a, sa, lanes, layout, cus, s);
}

size_t star_lds_bytes(int dim, int D, int M, int lanes) {
    return sizeof(float) * (size_t)(dim == 2 ? star_lds_floats<2>(D, M, lanes) : star_lds_floats<3>(D, M, lanes));
}

}  // namespace snk
