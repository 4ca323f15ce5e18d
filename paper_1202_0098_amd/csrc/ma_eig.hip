// Reduced generalised eigenproblems and column outputs (a6, a7), and the
// launcher of the kernel.
#include "ma_device.h"

namespace ma {

namespace {

// One column of the chunk per workgroup of CW * NG threads (nu <= RM <= CW).
// Thread t holds, for column t % CW, the rows (t / CW) * RM / NG + r of every
// nu x nu matrix in registers, so that each step of the factorisations is one
// rank-two update of RM / NG rows per thread against two vectors that go through LDS:
//   congruence  A = Lc^-1 H~ Lc^-T and G = Lc^-T together, one column of the
//               Cholesky factor of S~ = Lc Lc^T per step;
//   Householder A = Q T Q^T with G Q accumulated from the left;
//   implicit QL with shifts on T (Bowdler, Martin, Reinsch and Wilkinson,
//               Numer. Math. 11 (1968)), each plane rotation applied to two
//               columns of C = G Q (LDS, one lane per row), which ends as the
//               S~-orthonormal eigenvectors: there is no back substitution.
// Then v_a at row j, (S v_a)_j, the Ritz values in ascending order and the
// weights w_a = v_ja (S v_a)_j; then either the amplitudes v_ia v_ja at the
// pattern rows or, with a given chemical potential, rho_ij, pi_ij (Eqs. 13-14)
// and E_j, N_j (Eq. 17).
//
// What bounds it: instruction issue of the wavefront that runs the QL
// rotations (about 1,060 per column at nu = 30); the matrix cores and memory
// are idle.  Hence one wavefront per column up to nu = 32 (no barriers) and
// v_rsq_f64 with one third-order correction (within 2 ulp) in place of square roots
// and divisions.  Against the kernel below with its matrices in LDS and IEEE square
// roots: one column of nu = 30 197 us (553 us), 4,000 of them 604 us (1,462 us),
// one of nu = 16 67 us (189 us).
constexpr int kEigWaves = 3;   // waves per SIMD that the registers leave room for

template <int CW, int NG, int RM>
__global__ void __launch_bounds__(CW * NG, kEigWaves) k_eig(DevSystem S, DevJob J)
{
    constexpr int RPG = RM / NG, NT = CW * NG, NWV = NT / 64, LDZ = RM + 1;
    static_assert(RPG % 2 == 0 && RM % 16 == 0 && RM <= CW && (NT == 64 || CW == 64),
                  "one wavefront, or one per row group");
    // columns of C, LDZ apart, and (d, e) of T, each after one entry that a
    // sweep's last prefetch reads
    __shared__ double Zm[(CW + 1) * LDZ];
    __shared__ double2 de_[CW + 1 + 64];     // 64 more: where the lanes that do not keep T write
    double *Z = Zm + LDZ;
    double2 *de = de_ + 1;
    __shared__ double xs[CW], ys[CW], gs[CW], lv[CW], bv_[CW], gv[CW];
    __shared__ double ev[CW], vj[CW], fw[CW];
    __shared__ double part[NWV > 1 ? 2 * NG * CW : 1];
    __shared__ int rank[CW], s_status;
    const int nu = J.nu, o = S.o;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int col = tid % CW, grp = tid / CW, row0 = grp * RPG;

    // sum of a value over the row groups, for every column (two at a time)
    auto group_sum = [&](double &a, double &b) __attribute__((always_inline)) {
        if constexpr (NWV == 1) {
            a = sum_across<CW>(a);
            b = sum_across<CW>(b);
        } else {
            __syncthreads();
            part[grp * CW + col] = a;
            part[(NG + grp) * CW + col] = b;
            __syncthreads();
            a = b = 0.0;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                a += part[g * CW + col];
                b += part[(NG + g) * CW + col];
            }
        }
    };

    const int s = blockIdx.x;
    const int c = J.order[J.c0 + s];
    const double *mid = J.mid + (int64_t)s * J.mid_stride;
    const double *Up = mid + 2 * (int64_t)nu * nu;
    int32_t *st = J.stats + (int64_t)c * kStats;
    int L = st[3] == 0 ? st[0] : 0;
    int status = 0;
    double A[RPG], B[RPG], G[RPG];
#pragma unroll
    for (int r = 0; r < RPG; ++r) {
        const int i = row0 + r;
        const bool in = i < L && col < L;
        const int e = in ? i * nu + col : 0, t = in ? col * nu + i : 0;
        const double h = 0.5 * (mid[e] + mid[t]);
        const double m = 0.5 * (mid[nu * nu + e] + mid[nu * nu + t]);
        A[r] = in ? h : 0.0;
        B[r] = in ? m : 0.0;
        G[r] = i == col ? 1.0 : 0.0;
    }

    // the columns past the rows are zero throughout
    if (RM < CW && tid >= RM && tid < CW) xs[tid] = ys[tid] = gs[tid] = 0.0;
    // Congruence.  With l the column k of the Cholesky factor (l_k set to
    // lk - 1) and a = A e_k / lk, b = a - (alpha / 2) l:
    // A -= l b^T + b l^T and G -= g l^T scale and eliminate row and column
    // k at once (the diagonal of S~ is 1 to rounding: its vectors are
    // S-normalised).
    for (int k = 0; k < L; ++k) {
        if (col == k) {
#pragma unroll
            for (int r = 0; r < RPG; ++r) {
                xs[row0 + r] = B[r];
                ys[row0 + r] = A[r];
                gs[row0 + r] = G[r];
            }
        }
        __syncthreads();
        double dk = xs[k];
        const bool bad = !(dk >= DBL_MIN);
        status = bad ? -4 : status;
        dk = bad ? 1.0 : dk;
        const double rl = rsqrt_fast(dk), lk = dk * rl;
        const double alpha = ys[k] * rl * rl;
        const double lj = col > k ? xs[col] * rl : col == k ? lk - 1.0 : 0.0;
        const double bj = col == k ? alpha + 0.5 * alpha * lj : ys[col] * rl - 0.5 * alpha * lj;
        if (grp == 0) {
            lv[col] = lj;
            bv_[col] = bj;
            gv[col] = gs[col] * rl;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RPG; ++r) {
            const double li = lv[row0 + r];
            A[r] -= li * bj + bv_[row0 + r] * lj;
            B[r] -= li * lj;
            G[r] -= gv[row0 + r] * lj;
        }
    }
    // G = Lc^-T, one row per lane from here on
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RPG; ++r) Z[col * LDZ + row0 + r] = G[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RPG; ++r) G[r] = Z[(row0 + r) * LDZ + col];
    __syncthreads();

    // Householder reduction: step k reflects x = A[k+1.., k] onto
    // alpha e_1 with P = I - v v^T / h, v = x - alpha e_1, h = |v|^2 / 2
    double e_own = 0.0;   // lane k: the sub-diagonal entry k
    for (int k = 0; k + 2 < L; ++k) {
        if (col == k) {
#pragma unroll
            for (int r = 0; r < RPG; ++r) xs[row0 + r] = A[r];
        }
        __syncthreads();
        const double xj = col > k ? xs[col] : 0.0;
        const double x0 = xs[k + 1];
        const double sig = sum_within<CW>(xj * xj);
        const bool reflect = sig >= DBL_MIN;
        const double sg = reflect ? sig : 1.0;
        const double nrm = sg * rsqrt_fast(sg);
        const double alpha = x0 >= 0.0 ? -nrm : nrm;
        const double rh = reflect ? rcp_fast(sg - x0 * alpha) : 0.0;
        e_own = col == k ? (reflect ? alpha : x0) : e_own;
        const double vcol = reflect ? (col == k + 1 ? x0 - alpha : xj) : 0.0;
        if (grp == 0) lv[col] = vcol;
        __syncthreads();
        double v[RPG], pj = 0.0, t = 0.0;
#pragma unroll
        for (int r = 0; r < RPG; ++r) v[r] = lv[row0 + r];
#pragma unroll
        for (int r = 0; r < RPG; ++r) {
            pj += A[r] * v[r];
            t += G[r] * v[r];
        }
        group_sum(pj, t);
        pj *= rh;
        t *= rh;
        const double K = 0.5 * rh * sum_within<CW>(vcol * pj);
        const double qj = pj - K * vcol;
        if (grp == 0) bv_[col] = qj;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RPG; ++r) {
            A[r] -= v[r] * qj + bv_[row0 + r] * vcol;
            G[r] -= t * v[r];
        }
    }
    // T into LDS, C = G Q column by column
    double diag = 0.0, last = 0.0;
#pragma unroll
    for (int r = 0; r < RPG; ++r) {
        diag = row0 + r == col ? A[r] : diag;
        last = row0 + r == L - 1 ? A[r] : last;
        if (RM == CW || col < RM) Z[(row0 + r) * LDZ + col] = G[r];
    }
    if (col >= row0 && col < row0 + RPG) de[col].x = diag;
    if (col == L - 2 && L - 1 >= row0 && L - 1 < row0 + RPG) de[col].y = last;
    if (grp == 0 && col + 2 < L) de[col].y = e_own;
    if (grp == 0 && col >= L - 1) de[col].y = 0.0;
    if (tid == 0) s_status = status;
    __syncthreads();

    // Implicit QL sweeps by the first wavefront.  For the leading
    // unreduced block [l, m] (e_m negligible against its diagonal
    // neighbours), a shift from the 2 x 2 at l, then plane rotations
    // chasing the bulge from m up to l.  At most 64 sweeps per eigenvalue.
    // Column i of C stays in a register between the rotations (i, i + 1)
    // and (i - 1, i); d, e and the column of the next rotation are read
    // one rotation ahead.  The loop is one wavefront's instruction issue
    // (about 45 per rotation), so it has no branch inside: f = g = 0 takes
    // the identity as its rotation, the lanes past the rows repeat some, and d, e
    // are written by lane 0 while the others write to places of their own.
    if (wv == 0) {
        const int rl = lane % RM;
        const int own = lane == 0 ? 1 : 0;
        for (int l = 0; l < L && status == 0; ++l) {
            int sweeps = 0;
            for (;;) {
                wave_sync();
                bool small = lane == L - 1;
                if (lane >= l && lane < L - 1) {
                    const double2 t0 = de[lane];
                    small = fabs(t0.y) <= DBL_EPSILON * (fabs(t0.x) + fabs(de[lane + 1].x));
                }
                const unsigned long long msk = __ballot(small) >> l;
                const int m = l + __ffsll((long long)msk) - 1;
                if (m == l) break;
                if (++sweeps > 64) {
                    status = -5;
                    break;
                }
                const double2 tl = de[l];
                const double dm = de[m].x, u = de[l + 1].x - tl.x;
                double2 t_i = de[m - 1];
                double z_i1 = Z[m * LDZ + rl], z_i = Z[(m - 1) * LDZ + rl];
                // eigenvalue of the 2 x 2 nearer to d_l
                const double e2 = 2.0 * tl.y * tl.y;
                const double w2 = fma(u, u, 2.0 * e2);
                const double w = w2 < DBL_MIN ? 0.0 : w2 * rsqrt_fast(w2);
                const double den = u >= 0.0 ? u + w : u - w;
                double g = dm - tl.x + (fabs(den) < DBL_MIN ? 0.0 : e2 * rcp_fast(den));
                double sn = 1.0, cs = 1.0, p = 0.0, d_i1 = dm;
                double *zp = Z + m * LDZ + rl;
                const double2 *rp = de + m - 2;
                double2 *wp = own ? de + m : de + CW + lane;
                for (int i = m - 1; i >= l; --i) {
                    const double2 t_n = *rp--;
                    const double z_n = zp[-2 * LDZ];
                    const double f = sn * t_i.y, b = cs * t_i.y;
                    const double r2 = fma(f, f, g * g);
                    const bool none = r2 < DBL_MIN;
                    const double ir = rsqrt_fast(r2);
                    sn = none ? 0.0 : f * ir;
                    cs = none ? 1.0 : g * ir;
                    g = d_i1 - p;
                    const double rr = fma(t_i.x - g, sn, 2.0 * cs * b);
                    p = sn * rr;
                    *wp = make_double2(g + p, none ? 0.0 : r2 * ir);
                    wp -= own;
                    g = fma(cs, rr, -b);
                    *zp = fma(sn, z_i, cs * z_i1);
                    z_i1 = fma(cs, z_i, -sn * z_i1);
                    zp -= LDZ;
                    z_i = z_n;
                    d_i1 = t_i.x;
                    t_i = t_n;
                }
                *zp = z_i1;
                *wp = make_double2(tl.x - p, g);
                de[m].y = 0.0;
            }
        }
        wave_sync();
        if (lane == 0) s_status = status;
    }
    __syncthreads();
    status = s_status;
    if (status != 0) {
        L = 0;
        if (tid == 0) {
            st[0] = 0;
            st[3] = status;
            atomicMin(J.fail, c);
        }
    }
    // ascending ranks; v_a and (S v_a) at row j (the rows of a thread's
    // group, then over the groups)
    double v1 = 0.0, v2 = 0.0;
    {
        double u1[RPG], u2[RPG];
#pragma unroll
        for (int r = 0; r < RPG; ++r) {
            const int m = row0 + r < L ? row0 + r : 0;
            u1[r] = Up[m];
            u2[r] = Up[nu + m];
        }
#pragma unroll
        for (int r = 0; r < RPG; ++r) {
            const double cma = row0 + r < L ? Z[col * LDZ + row0 + r] : 0.0;
            v1 += u1[r] * cma;
            v2 += u2[r] * cma;
        }
    }
    group_sum(v1, v2);
    double *eps_o = J.eps + (int64_t)c * nu, *wts_o = J.wts + (int64_t)c * nu;
    if (grp == 0 && col < nu) {
        if (col < L) {
            int rk = 0;
            const double va = de[col].x;
#pragma unroll 8
            for (int b = 0; b < L; ++b) {
                const double vb = de[b].x;
                rk += vb < va || (vb == va && b < col) ? 1 : 0;
            }
            ev[col] = va;
            vj[col] = v1;
            rank[col] = rk;
            eps_o[rk] = va;
            wts_o[rk] = v1 * v2;
        } else {
            eps_o[col] = NAN;
            wts_o[col] = 0.0;
        }
    }
    __syncthreads();
    const int j = J.cols[c];
    const int At = j / o, r = j - At * o;
    const int64_t kb0 = S.blk_ptr[At];
    const int npat = (int)(S.blk_ptr[At + 1] - kb0) * o;
    if (!J.direct) {
        // V at the pattern rows on the FP64 matrix cores: 16 x 16 tiles of
        // (basis rows of the chunk buffer, npat x L) x (C, L x L, LDS), with
        // v_mfma_f64_16x16x4f64: lane l feeds A[l%16][l/16], B[l/16][l%16]
        // and receives D[4 j + l/16][l%16]
        double *amp = reinterpret_cast<double *>(J.amp) + J.amp_off[c];
        const int nrt = (npat + 15) >> 4, nct = (nu + 15) >> 4;
        const int kq = lane >> 4, l16 = lane & 15;
        for (int mt = wv; mt < nrt; mt += NWV) {
            const int arow = mt * 16 + l16;
            // this lane's basis-row operands, loaded together
            double avs[RM / 4];
#pragma unroll
            for (int k4 = 0; k4 < RM / 4; ++k4) {
                const int kk = 4 * k4 + kq;
                const bool in = arow < npat && kk < L;
                const double uv = Up[in ? (2 + arow) * nu + kk : 0];
                avs[k4] = in ? uv : 0.0;
            }
            for (int ct = 0; ct < nct; ++ct) {
                const int bcol = ct * 16 + l16;
                dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int k4 = 0; k4 < RM / 4; ++k4) {
                    const int kk = 4 * k4 + kq;
                    const double zv = Z[(bcol < RM ? bcol : 0) * LDZ + kk];
                    const double cv = bcol < L && kk < L ? zv : 0.0;
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(avs[k4], cv, acc, 0, 0, 0);
                }
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int tr = mt * 16 + 4 * jj + kq;
                    if (tr < npat && bcol < nu) {
                        if (bcol < L) amp[tr * nu + rank[bcol]] = acc[jj] * vj[bcol];
                        else amp[tr * nu + bcol] = 0.0;
                    }
                }
            }
        }
    } else {
        // rho_i = sum_m u_m[i] y_m with y = C (f v_j), and pi with f eps v_j
        if (grp == 0 && col < L) fw[col] = fermi((ev[col] - J.mu) / J.kT) * vj[col];
        __syncthreads();
        double y = 0.0, yp = 0.0;
#pragma unroll
        for (int r2 = 0; r2 < RPG; ++r2) {
            const int a = row0 + r2;
            const double z = a < L ? Z[a * LDZ + col] * fw[a] : 0.0;
            y += z;
            yp += a < L ? z * ev[a] : 0.0;
        }
        group_sum(y, yp);
        if (grp == 0) {
            lv[col] = y;
            bv_[col] = yp;
        }
        __syncthreads();
        double ep = 0.0, np_ = 0.0;
        for (int tt = tid; tt < npat; tt += NT) {
            double sr = 0.0, sp = 0.0;
#pragma unroll 16
            for (int m = 0; m < L; ++m) {
                const double um = Up[(2 + tt) * nu + m];
                sr += um * lv[m];
                sp += um * bv_[m];
            }
            const int64_t slot = ((kb0 + tt / o) * o + r) * o + (tt % o);
            if (J.rho) J.rho[slot] = sr;
            if (J.pi) J.pi[slot] = sp;
            ep += sr * S.Hd[slot];
            np_ += sr * S.Sd[slot];
        }
        ep = sum_within<64>(ep);
        np_ = sum_within<64>(np_);
        if constexpr (NWV > 1) {
            if (lane == 0) {
                xs[wv] = ep;
                ys[wv] = np_;
            }
            __syncthreads();
            ep = np_ = 0.0;
            for (int w = 0; w < NWV; ++w) {
                ep += xs[w];
                np_ += ys[w];
            }
        }
        if (tid == 0) {
            J.Ecol[c] = ep;
            J.Ncol[c] = np_;
        }
    }
}

// The same, for amplitudes kept in FP32 (mixed modes, chemical potential
// bisected).  A stored amplitude moves by an FP32 ulp (6e-8) where the last FP64
// bit before its rounding changes, so this kernel keeps one fixed order of
// every FP64 sum; the kernel above, whose sums are grouped otherwise, takes the
// cases where nothing is rounded to FP32 afterwards.  One wavefront per column of the
// chunk, everything in LDS:
//   1/2 (X + X^T) -> H~, S~; Cholesky S~ = Lc Lc^T (right-looking);
//   A = Lc^-1 H~ Lc^-T (two right-looking triangular solves, a lane per column);
//   Householder reduction A = Q T Q^T, Q accumulated backwards; implicit QL;
//   C = Lc^-T Z.
// Every lane runs the scalar recurrences of the QL sweeps redundantly, so they
// need no broadcasts.  Bound by instruction issue of the nine wavefronts that LDS
// lets a compute unit hold at nu = 30: 62,208 columns 15.9 ms; with eight, 17.5; with
// lanes masked in the rotation loop too, 20.5, and with one lane per column in the
// updates, 22.0.
__global__ void __launch_bounds__(64) k_eig_f32(DevSystem S, DevJob J)
{
    extern __shared__ double smem[];
    const int nu = J.nu;
    // Two nu x nu matrices in LDS (A, and Z column-major); the Cholesky
    // factor of S~ lives in the Z area until Z is needed, waits in the S~
    // slot of the chunk buffer meanwhile, and comes back for C = Lc^-T Z.
    double *A = smem, *Z = smem + nu * nu, *B = Z;
    double *ev = smem + 2 * nu * nu, *vj = ev + nu, *svj = vj + nu;
    double *hh = svj + nu, *ee = hh + nu, *rd = ee + nu;
    double *upj = rd + nu;   // 2 nu
    int *rank = reinterpret_cast<int *>(upj + 2 * nu);
    __shared__ double hv[kMaxNu];   // current Householder vector (separate objects: the
    __shared__ double hq[kMaxNu];   // compiler may keep their loads ahead of A's stores)
    const int lane = threadIdx.x;
    const int o = S.o;
    for (int s = blockIdx.x; s < J.cn; s += gridDim.x) {
        const int c = J.order[J.c0 + s];
        double *mid = J.mid + (int64_t)s * J.mid_stride;
        const double *Up = mid + 2 * (int64_t)nu * nu;
        int32_t *st = J.stats + (int64_t)c * kStats;
        int L = st[3] == 0 ? st[0] : 0;
        int status = 0;
        // up to 32 columns: two lanes per column, which take turns along its rows
        // in the updates (a sum of products stays one lane's)
        const bool two = L <= 32;
        const int c0 = two ? lane & 31 : lane, r0 = two ? lane >> 5 : 0, dr = two ? 2 : 1;
#pragma unroll 4
        for (int e = lane; e < L * L; e += 64) {
            const int i = e / L, k = e - i * L;
            A[e] = 0.5 * (mid[i * nu + k] + mid[k * nu + i]);
            B[e] = 0.5 * (mid[nu * nu + i * nu + k] + mid[nu * nu + k * nu + i]);
        }
        // basis rows at j: u_m[j] and (S u_m)[j]
        for (int m = lane; m < L; m += 64) {
            upj[m] = Up[m];
            upj[nu + m] = Up[nu + m];
        }
        __syncthreads();

        // Cholesky S~ = Lc Lc^T in the lower triangle of B
        for (int k = 0; k < L; ++k) {
            double dk = B[k * L + k];
            if (!(dk > 0.0)) {
                status = -4;
                dk = 1.0;
            }
            const double lk = sqrt(dk), rl = 1.0 / lk;
            for (int i = k + 1 + lane; i < L; i += 64) B[i * L + k] *= rl;
            __syncthreads();
            const int j = k + 1 + c0;
            if (j < L) {
                const double bjk = B[j * L + k];
                #pragma unroll 4
                for (int i = j + r0; i < L; i += dr) B[i * L + j] -= B[i * L + k] * bjk;
            }
            if (lane == 0) {
                B[k * L + k] = lk;
                rd[k] = rl;
            }
            __syncthreads();
        }
        // A = Lc^-1 H~ Lc^-T in place: W = Lc^-1 A (a lane per column), then
        // A = Lc^-1 W^T
        for (int pass = 0; pass < 2; ++pass) {
            for (int k = 0; k < L; ++k) {
                if (c0 < L) {
                    const double ak = A[k * L + c0] * rd[k];
                    #pragma unroll 4
                    for (int i = k + 1 + r0; i < L; i += dr) A[i * L + c0] -= B[i * L + k] * ak;
                    if (r0 == 0) A[k * L + c0] = ak;
                }
                wave_sync();
            }
            __syncthreads();
            if (pass == 0) {
                for (int e = lane; e < L * L; e += 64) {
                    const int i = e / L, k = e - i * L;
                    if (i < k) {
                        const double x = A[i * L + k];
                        A[i * L + k] = A[k * L + i];
                        A[k * L + i] = x;
                    }
                }
                __syncthreads();
            }
        }
        // the factor waits in the S~ slot of the chunk buffer (read above,
        // not read again) while Z takes its place
        for (int e = lane; e < L * L; e += 64) mid[nu * nu + e] = B[e];
        __syncthreads();
        for (int e = lane; e < L * L; e += 64) {
            const int i = e / L, k = e - i * L;
            if (i < k) {
                const double v = 0.5 * (A[i * L + k] + A[k * L + i]);
                A[i * L + k] = v;
                A[k * L + i] = v;
            }
        }
        __syncthreads();

        // Householder reduction to tridiagonal form.  Step k reflects
        // x = A[k+1.., k] onto alpha e_1 with P = I - v v^T / h,
        // v = x - alpha e_1, h = |v|^2 / 2; v stays in column k below the
        // diagonal, h in hh[k], alpha is the sub-diagonal ee[k].
        for (int k = 0; k + 2 < L; ++k) {
            const int i = k + 1 + lane;
            const double xi = i < L ? A[i * L + k] : 0.0;
            const double sig = wave_sum(xi * xi);
            const double x0 = A[(k + 1) * L + k];
            double alpha = x0, h = 0.0;
            if (sig > 0.0) {
                alpha = x0 >= 0.0 ? -sqrt(sig) : sqrt(sig);
                h = sig - x0 * alpha;
            }
            if (lane == 0) {
                ee[k] = alpha;
                hh[k] = h;
            }
            if (h > 0.0) {
                // v = x - alpha e_1, kept in column k and in hv
                const double vi = (i == k + 1) ? x0 - alpha : xi;
                if (i < L) {
                    hv[i] = vi;
                    A[i * L + k] = vi;
                }
                __syncthreads();
                // p = A' v / h, K = v^T p / (2 h), q = p - K v (a lane per column j)
                const int j = k + 1 + lane;
                double pj = 0.0, vjj = 0.0;
                if (j < L) {
                    #pragma unroll 4
                    for (int ii = k + 1; ii < L; ++ii) pj += A[ii * L + j] * hv[ii];
                    pj /= h;
                    vjj = hv[j];
                }
                const double K = wave_sum(vjj * pj) / (2.0 * h);
                const double qj = pj - K * vjj;
                if (j < L) hq[j] = qj;
                __syncthreads();
                // A' -= v q^T + q v^T
                const int jc = k + 1 + c0;
                if (jc < L) {
                    const double qc = hq[jc], vc = hv[jc];
                    #pragma unroll 4
                    for (int ii = k + 1 + r0; ii < L; ii += dr)
                        A[ii * L + jc] -= hv[ii] * qc + hq[ii] * vc;
                }
            }
            __syncthreads();
        }
        for (int i = lane; i < L; i += 64) ev[i] = A[i * L + i];
        if (lane == 0 && L >= 2) ee[L - 2] = A[(L - 1) * L + L - 2];
        if (lane == 0 && L >= 1) ee[L - 1] = 0.0;
        // Z = P_0 P_1 ... P_{L-3} (column-major), accumulated from the last
        // reflector; P_k leaves columns 0..k unchanged
        for (int e = lane; e < L * L; e += 64) Z[e] = (e / L == e % L) ? 1.0 : 0.0;
        __syncthreads();
        for (int k = L - 3; k >= 0; --k) {
            const double h = hh[k];
            if (!(h > 0.0)) continue;
            const int cc = k + 1 + c0;
            if (cc < L) {
                double t = 0.0;
                #pragma unroll 4
                for (int i = k + 1; i < L; ++i) t += A[i * L + k] * Z[cc * L + i];
                t /= h;
                #pragma unroll 4
                for (int i = k + 1 + r0; i < L; i += dr) Z[cc * L + i] -= A[i * L + k] * t;
            }
            wave_sync();
        }
        __syncthreads();

        // Implicit QL sweeps on (ev, ee).  For the leading unreduced block
        // [l, m] (ee[m] negligible against its diagonal neighbours), a shift
        // from the 2 x 2 at l, then plane rotations chasing the bulge from m
        // up to l.  At most 64 sweeps per eigenvalue.  The rotation loop is
        // software-pipelined: the entries of the next rotation are loaded one
        // rotation ahead, and the rotated column i stays in a register for the
        // next rotation (columns i + 1 are final once written).  No lane is masked
        // out: those past the rows repeat row 0, and those that do not keep T write
        // their entries to the idle Householder vectors.  Which products are
        // rounded before they are added is written out (p is, by the empty asm).
        const int rw = lane < L ? lane : 0, own = lane == 0 ? 1 : 0;
        for (int l = 0; l < L && status == 0; ++l) {
            int sweeps = 0;
            for (;;) {
                // m: the first k >= l with ee[k] negligible (L - 1 if none),
                // one lane per k
                bool small = lane == L - 1;
                if (lane >= l && lane < L - 1)
                    small = fabs(ee[lane]) <= DBL_EPSILON * (fabs(ev[lane]) + fabs(ev[lane + 1]));
                const unsigned long long msk =
                    __ballot(small) & ~((l > 0 ? (1ull << l) : 1ull) - 1ull);
                const int m = __ffsll((long long)msk) - 1;
                if (m == l) break;
                if (++sweeps > 64) {
                    status = -5;
                    break;
                }
                const double el = ee[l], dl0 = ev[l], dl1 = ev[l + 1], dm = ev[m];
                const double t0 = (dl1 - dl0) / (2.0 * el);
                const double r0 = sqrt(t0 * t0 + 1.0);
                double g = dm - dl0 + el / (t0 + (t0 >= 0.0 ? r0 : -r0));
                double sn = 1.0, cs = 1.0, p = 0.0;
                bool underflow = false;
                double e_i = ee[m - 1], d_i = ev[m - 1], d_i1 = dm;
                double *zp = Z + m * L + rw;
                double z_i1 = zp[0], z_i = zp[-L];
                double *ep = lane == 0 ? ee + m : hv + lane, *dp = lane == 0 ? ev + m : hq + lane;
                for (int i = m - 1; i >= l; --i) {
                    // (the last prefetch reads one entry below, whatever lies there)
                    const double e_n = ee[i - 1], d_n = ev[i - 1], z_n = zp[-2 * L];
                    const double f = sn * e_i, b = cs * e_i;
                    const double r2 = fma(g, g, f * f);
                    if (__ballot(r2 == 0.0)) {
                        const double dnew = d_i1 - p;
                        if (lane == 0) {
                            ee[i + 1] = 0.0;
                            ev[i + 1] = dnew;
                            ee[m] = 0.0;
                        }
                        *zp = z_i1;
                        underflow = true;
                        break;
                    }
                    const double ir = rsqrt(r2);
                    sn = f * ir;
                    cs = g * ir;
                    g = d_i1 - p;
                    const double rr = fma(d_i - g, sn, 2.0 * cs * b);
                    p = sn * rr;
                    asm("" : "+v"(p));
                    *ep = r2 * ir;
                    *dp = g + p;
                    ep -= own;
                    dp -= own;
                    g = fma(cs, rr, -b);
                    const double zn1 = fma(sn, z_i, cs * z_i1);
                    const double zn0 = fma(cs, z_i, -(sn * z_i1));
                    *zp = zn1;
                    zp -= L;
                    z_i1 = zn0;
                    z_i = z_n;
                    e_i = e_n;
                    d_i1 = d_i;
                    d_i = d_n;
                }
                if (underflow) continue;
                *zp = z_i1;
                if (lane == 0) {
                    ev[l] = dl0 - p;
                    ee[l] = g;
                    ee[m] = 0.0;
                }
            }
        }
        __syncthreads();
        // ascending ranks of the eigenvalues
        for (int a = lane; a < L; a += 64) {
            int rk = 0;
            const double va = ev[a];
            #pragma unroll 4
            for (int bb = 0; bb < L; ++bb)
                if (ev[bb] < va || (ev[bb] == va && bb < a)) ++rk;
            rank[a] = rk;
        }
        // C = Lc^-T Z -> A (row-major), a lane per column; the factor back
        // in the Z area once Z is copied
        for (int a = lane; a < L; a += 64) {
            #pragma unroll 4
            for (int i = 0; i < L; ++i) A[i * L + a] = Z[a * L + i];
        }
        __syncthreads();
        for (int e = lane; e < L * L; e += 64) B[e] = mid[nu * nu + e];
        __syncthreads();
        for (int k = L - 1; k >= 0; --k) {
            if (c0 < L) {
                const double ck = A[k * L + c0] * rd[k];
                #pragma unroll 4
                for (int i = r0; i < k; i += dr) A[i * L + c0] -= B[k * L + i] * ck;
                if (r0 == 0) A[k * L + c0] = ck;
            }
            wave_sync();
        }
        __syncthreads();
        if (status != 0) {
            L = 0;
            if (lane == 0) {
                st[0] = 0;
                st[3] = status;
                atomicMin(J.fail, c);
            }
        }
        const double *C = A;
        // v_a and (S v_a) at row j (a lane per Ritz vector; the basis rows
        // are read at the same address by every lane)
        for (int a = lane; a < L; a += 64) {
            double v1 = 0.0, v2 = 0.0;
            #pragma unroll 4
            for (int m = 0; m < L; ++m) {
                const double cma = C[m * L + a];
                v1 += upj[m] * cma;
                v2 += upj[nu + m] * cma;
            }
            vj[a] = v1;
            svj[a] = v2;
        }
        __syncthreads();
        double *eps_o = J.eps + (int64_t)c * nu, *wts_o = J.wts + (int64_t)c * nu;
        for (int a = lane; a < nu; a += 64) {
            if (a < L) {
                eps_o[rank[a]] = ev[a];
                wts_o[rank[a]] = vj[a] * svj[a];
            } else {
                eps_o[a] = NAN;
                wts_o[a] = 0.0;
            }
        }
        const int j = J.cols[c];
        const int At = j / o, r = j - At * o;
        const int64_t kb0 = S.blk_ptr[At];
        const int npat = (int)(S.blk_ptr[At + 1] - kb0) * o;
        {
            // V at the pattern rows on the FP64 matrix cores: 16 x 16 tiles of
            // (basis rows of the chunk buffer, npat x L) x (C, L x L, LDS), with
            // v_mfma_f64_16x16x4f64: lane l feeds A[l%16][l/16], B[l/16][l%16]
            // and receives D[4 j + l/16][l%16]
            float *amp = reinterpret_cast<float *>(J.amp) + J.amp_off[c];
            const int nrt = (npat + 15) >> 4, nct = (nu + 15) >> 4;
            const int kq = lane >> 4, l16 = lane & 15;
            for (int mt = 0; mt < nrt; ++mt) {
                const int arow = mt * 16 + l16;
                // this lane's basis-row operands for the first 32 k, loaded together
                double avs[8];
#pragma unroll
                for (int st4 = 0; st4 < 8; ++st4) {
                    const int kk = 4 * st4 + kq;
                    avs[st4] = (arow < npat && kk < L) ? Up[(2 + arow) * nu + kk] : 0.0;
                }
              for (int ct = 0; ct < nct; ++ct) {
                const int bcol = ct * 16 + l16;
                dbl4 acc = {0.0, 0.0, 0.0, 0.0};
                for (int k0 = 0; k0 < L; k0 += 4) {
                    const int kk = k0 + kq;
                    const double av = k0 < 32 ? avs[(k0 >> 2) & 7]
                                      : (arow < npat && kk < L) ? Up[(2 + arow) * nu + kk] : 0.0;
                    const double bv = (bcol < L && kk < L) ? C[kk * L + bcol] : 0.0;
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
                }
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int tr = mt * 16 + 4 * jj + kq;
                    if (tr < npat && bcol < nu) {
                        if (bcol < L) amp[tr * nu + rank[bcol]] = (float)(acc[jj] * vj[bcol]);
                        else amp[tr * nu + bcol] = (float)0.0;
                    }
                }
              }
            }
        }
        __syncthreads();   // LDS is reused by the next column
    }
}

template <int CW, int NG, int RM = CW>
hipError_t launch_width(const DevSystem &S, const DevJob &J, hipStream_t st)
{
    hipLaunchKernelGGL((k_eig<CW, NG, RM>), dim3(J.cn), dim3(CW * NG), 0, st, S, J);
    return hipGetLastError();
}

}  // namespace

// Amplitudes in FP32: k_eig_f32.  Otherwise the smallest width that holds nu:
// one wavefront per column up to 32 (16 columns x 4 row groups, 32 x 2), two
// with 24 rows each up to 48 (12,004 columns of nu = 40: 5.7 ms, 7.0 with the four
// below: what every wavefront does for itself in a step, about 100 instructions,
// weighs as much as its rows), beyond that four with 16 rows each.
hipError_t launch_eig(const DevSystem &S, const DevJob &J, hipStream_t st)
{
    if (J.cn < 1) return hipSuccess;
    if (J.precision != 0 && !J.direct) {
        const size_t smem = sizeof(double) * (2 * (size_t)J.nu * J.nu + 8 * (size_t)J.nu) +
                            sizeof(int) * (size_t)J.nu;
        hipError_t e = hipFuncSetAttribute((const void *)k_eig_f32,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        const int grid = J.cn < (1 << 20) ? J.cn : (1 << 20);
        hipLaunchKernelGGL(k_eig_f32, dim3(grid), dim3(64), smem, st, S, J);
        return hipGetLastError();
    }
    if (J.nu <= 16) return launch_width<16, 4>(S, J, st);
    if (J.nu <= 32) return launch_width<32, 2>(S, J, st);
    if (J.nu <= 48) return launch_width<64, 2, 48>(S, J, st);
    return launch_width<64, 4>(S, J, st);
}

}  // namespace ma
