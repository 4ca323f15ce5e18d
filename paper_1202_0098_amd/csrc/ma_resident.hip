// Resident basis kernel k_basis_r: one column per workgroup, its whole basis
// in the registers of the workgroup (FP64, regions of at most 64 NW orbitals).
//
// The workspace kernel reads and writes every stored vector once per step
// through memory (about 4.8 MB per column of 480 orbitals at nu = 30), which
// bounds it.  A compute unit's registers hold 512 KB, a column's U (nu
// vectors of the region) 115 KB at that size, so here U stays on chip, twice:
//
//   * UA, the A operand of v_mfma_f64_4x4x4_4b over rows: lane l of wavefront
//     w holds vector 16 t + l % 16 at the rows 64 w + 16 (l / 16) .. + 15.  All
//     dots of a step are products over the wavefront's own 64 rows with up to
//     four right-hand vectors as columns of B; only the partial dots go
//     through LDS;
//   * UB, the B operand over vectors: lane l holds vector 4 q + l / 16 at the
//     rows 64 w + 16 r + l % 16.  Up to four linear combinations of the stored
//     vectors (rows of A) are products over all of them, and an exchange
//     between lanes hands each thread its own row.
//
//   S U and H U are not stored.  With p the pending vector (projected once) a
//   step forms S p, H p and S c (c its next candidate), and takes
//       a = U^T S p, b = U^T S c, k = U^T H p,
//   from which, with u = (p - U a) / beta, the column of the pair follows:
//       U^T H u = (k - H~ a) / beta,
//       u^T H u = (p^T H p - a.k - a.(k - H~ a)) / beta^2,
//   exactly the pair of the finished vectors (H~ is the pair so far), and
//   U^T S u = 0, u^T S u = 1 to rounding: S~ = I.
//   The Euclidean chain t_k on s_j, which does not depend on U, runs ahead
//   during block 1 and is complete before block 2 takes its seeds from it.
//   t_k waits in the slot of basis vector p + k, which replaces it (U and the
//   chain together never need more than nu slots), and in LDS by rows, where an
//   operator product reads it as a seed.
//
// What bounds it: instruction issue (two wavefronts per SIMD, about a thousand
// instructions per step and wavefront) and the round trips between phases; its
// memory traffic is the operator and the outputs.  Measured against the workspace
// kernel, nu = 30, 480 orbitals: one column 187 us (383), 4,000 columns 3.0 ms
// (4.5), 16,384 columns 12.1 ms (17.0); nu = 16, 256 orbitals: one column 76 us (132).
// A form with the vectors spread over the wavefronts (partial combinations
// through LDS) and one with U row-owned and scalar-broadcast coefficients took
// 463 and 278 us per column.
//
// Otherwise the arithmetic is the workspace kernel's: classical Gram-Schmidt
// twice with the second pass delayed into the next step, breakdown on beta
// against the candidate's norm rebuilt from both passes (Eqs. 6-9, Sec. 2).
#include "ma_device.h"

namespace ma {

namespace {

// The thread's row of the region operator: its blocks are k0 .. k1 of the
// staged index.  The values of the first KEEP blocks are loaded together, before
// the vectors they meet are complete, and S's are held for a step's second
// product; absent blocks point at the zero rows past the vectors' end, so that a
// product needs no selects.  KEEP = 2: each block of both operators holds 32
// registers beside the 128 of U; two take the last of them and 64 bytes per lane of
// scratch, three or more spill more than they save (a 4,000-column solve 4.68 ms, 4.73
// with three, 6.79 with all five of a crystal's row).
template <int O>
struct Row {
    static constexpr int KEEP = 2;
    int k0, k1, ri, zero;
    const int2 *sblk;
    int xo[KEEP];            // column atoms of the kept blocks
    __device__ __forceinline__ int64_t base(int kb) const
    {
        kb = kb < k1 ? kb : k0;
        return (int64_t)sblk[kb].y * (O * O) + ri * O;
    }
    __device__ __forceinline__ bool more() const { return k1 - k0 > KEEP; }
};

// the O entries of a staged vector that belong to a block's column atom
template <int O>
__device__ __forceinline__ void entries(const double *x, int atom, double (&v)[O])
{
    static_assert(O % 2 == 0, "pairs");
#pragma unroll
    for (int c = 0; c < O; c += 2) {
        const double2 w = *reinterpret_cast<const double2 *>(x + atom * O + c);
        v[c] = w.x;
        v[c + 1] = w.y;
    }
}

// y += S x over the row's blocks past the kept ones
template <int O>
__device__ __forceinline__ void spmv_s_rest(const DevSystem &S, const Row<O> &w, const double *x,
                                            double &y)
{
    for (int kb = w.k0 + Row<O>::KEEP; kb < w.k1; ++kb) {
        const int64_t b = w.base(kb);
        double sv[O], v[O];
#pragma unroll
        for (int c = 0; c < O; ++c) sv[c] = S.Sd[b + c];
        entries<O>(x, w.sblk[kb].x, v);
#pragma unroll
        for (int c = 0; c < O; ++c) y += sv[c] * v[c];
    }
}

// the row's values in the kept blocks
template <int O>
__device__ __forceinline__ void load_kept(const double *__restrict__ M, const Row<O> &w,
                                          double (&v)[Row<O>::KEEP][O])
{
#pragma unroll
    for (int k = 0; k < Row<O>::KEEP; ++k) {
        const int64_t b = w.base(w.k0 + k);
#pragma unroll
        for (int c = 0; c < O; ++c) v[k][c] = M[b + c];
    }
}

// S x, with the kept values in sm
template <int O>
__device__ __forceinline__ double spmv_s(const DevSystem &S, const Row<O> &w,
                                         const double (&sm)[Row<O>::KEEP][O], const double *x)
{
    double y = 0.0;
#pragma unroll
    for (int k = 0; k < Row<O>::KEEP; ++k) {
        double v[O];
        entries<O>(x, w.xo[k], v);
#pragma unroll
        for (int c = 0; c < O; ++c) y += sm[k][c] * v[c];
    }
    if (w.more()) spmv_s_rest<O>(S, w, x, y);
    return y;
}

// ha = H xa, sa = S xa and third = M3 xb with M3 = S (THIRD_S) or H
template <int O, bool THIRD_S>
__device__ __forceinline__ void spmv3(const DevSystem &S, const Row<O> &w,
                                      const double (&hm)[Row<O>::KEEP][O],
                                      const double (&sm)[Row<O>::KEEP][O], const double *xa,
                                      const double *xb, double &ha, double &sa, double &third)
{
#pragma unroll
    for (int k = 0; k < Row<O>::KEEP; ++k) {
        double va[O], vb[O];
        entries<O>(xa, w.xo[k], va);
        entries<O>(xb, w.xo[k], vb);
#pragma unroll
        for (int c = 0; c < O; ++c) {
            ha += hm[k][c] * va[c];
            sa += sm[k][c] * va[c];
            third += (THIRD_S ? sm[k][c] : hm[k][c]) * vb[c];
        }
    }
    if (w.more())
        for (int kb = w.k0 + Row<O>::KEEP; kb < w.k1; ++kb) {
            const int64_t b = w.base(kb);
            double hv[O], sv[O], va[O], vb[O];
#pragma unroll
            for (int c = 0; c < O; ++c) {
                hv[c] = S.Hd[b + c];
                sv[c] = S.Sd[b + c];
            }
            entries<O>(xa, w.sblk[kb].x, va);
            entries<O>(xb, w.sblk[kb].x, vb);
#pragma unroll
            for (int c = 0; c < O; ++c) {
                ha += hv[c] * va[c];
                sa += sv[c] * va[c];
                third += (THIRD_S ? sv[c] : hv[c]) * vb[c];
            }
        }
}

// Sum over the workgroup: one barrier (the caller alternates the scratch, so
// that the next sum does not overwrite values still being read).
template <int NW>
__device__ __forceinline__ double sum_wg(double v, double *scratch)
{
    v = sum_within<64>(v);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) s += scratch[k];
    return s;
}

// Inner CG (a3) in FP64 for one row per thread: inner_cg's iteration with the
// row's values of S in registers.
template <int O, int NW>
__device__ void row_cg(const DevSystem &S, const DevJob &J, const Col &g, const Row<O> &w, int c,
                       double *xs, double *scratch, double &x, int &iters, int &nres, int &status,
                       int &start)
{
    const int tid = threadIdx.x, n = g.n, nout = kNbOut * O;
    const bool row = tid < n;
    const double ej = tid == g.jl ? 1.0 : 0.0;
    iters = nres = status = start = 0;
    x = 0.0;
    if (J.x0) {
        // predicted coefficients on the orbitals of the kNbOut nearest atoms
        xs[tid] = 0.0;
        __syncthreads();
        for (int e = tid; e < nout; e += 64 * NW) {
            const int k = e / O, cc = e - k * O;
            const int la = S.out_loc[(int64_t)g.A * kNbOut + k];
            if (la >= 0) xs[la * O + cc] = (double)J.x0[(int64_t)c * nout + e];
        }
        __syncthreads();
        x = xs[tid];
        start = 1;
        __syncthreads();
    }
    if (J.x0full) {
        // a start on the whole region (the kept s_j of an earlier solve)
        if (row) x = J.x0full[(int64_t)c * S.nmax + tid];
        start = 3;
    }
    double sm[Row<O>::KEEP][O];
    load_kept<O>(S.Sd, w, sm);
    auto apply = [&](double v) __attribute__((always_inline)) {
        xs[tid] = v;
        __syncthreads();
        return spmv_s<O>(S, w, sm, xs);
    };
    int flip = 0;
    auto total = [&](double v) __attribute__((always_inline)) {
        flip ^= NW;
        return sum_wg<NW>(v, scratch + flip);
    };
    const double tol2 = J.cg_tol * J.cg_tol;
    double r = ej, rho2 = 1.0;   // zero start: the residual is e_j itself
    if (start) {
        r = ej - apply(x);
        rho2 = total(r * r);
        ++nres;
        if (!(rho2 < 1.0)) {
            // the residual judge rejects the given start: zero start
            start += 1;
            x = 0.0;
            r = ej;
            rho2 = 1.0;
        }
    }
    bool converged = false;
    for (int restart = 0; restart <= 3 && !converged && status == 0; ++restart) {
        double p = r;
        for (int k = 0; k < n && uniform(rho2 > tol2); ++k) {
            const double q = apply(p);
            const double pq = total(p * q);
            if (uniform(!(pq > 0.0))) {
                status = -4;
                break;
            }
            const double alpha = rho2 / pq;
            x += alpha * p;
            r -= alpha * q;
            const double rn = total(r * r);
            p = r + (rn / rho2) * p;
            rho2 = rn;
            ++iters;
        }
        if (status) break;
        // judge on the true residual
        r = ej - apply(x);
        rho2 = total(r * r);
        ++nres;
        if (uniform(rho2 <= tol2)) converged = true;
    }
    if (status == 0 && !converged) status = -5;
    if (J.sj_store && status == 0) {
        // keep s_j for a later solve (MA_START_PREVIOUS)
        const int64_t jg = J.cols[c];
        if (row) J.sj_store[jg * S.nmax + tid] = x;
        if (tid == 0) J.sj_have[jg] = 1;
    }
    if (J.sj_near) {
        // s_j on the orbitals of the kNbOut nearest atoms (training targets)
        __syncthreads();
        xs[tid] = x;
        __syncthreads();
        for (int e = tid; e < nout; e += 64 * NW) {
            const int k = e / O, cc = e - k * O;
            const int la = S.out_loc[(int64_t)g.A * kNbOut + k];
            J.sj_near[(int64_t)c * nout + e] = (status == 0 && la >= 0) ? (float)xs[la * O + cc] : 0.0f;
        }
    }
    __syncthreads();
}

constexpr int kRhs = 5;   // right-hand vectors of a step's dots: S p, S c, H p, z, H z

// doubles of LDS besides the region index (q: length of the chain)
template <int NW, int TILES>
__host__ __device__ constexpr int64_t resident_doubles(int q)
{
    constexpr int64_t nt = 64 * NW, ld = nt + 8, m = 16 * TILES;
    return (6 + q) * ld + NW * (kRhs * m + 8) + 5 * m + 8 + m * (m + 1) + m + NW + nt / 4;
}

enum { kNoCand = 0, kBlock1 = 1, kSeed = 2 };

// x[r] of lane row c (l / 16 = c) to x[c] of lane row r
__device__ __forceinline__ void transpose4(double (&x)[4])
{
    swap32(x[0], x[2]);
    swap32(x[1], x[3]);
    swap16(x[0], x[1]);
    swap16(x[2], x[3]);
}

template <int O, int NW, int TILES>
__global__ void __launch_bounds__(64 * NW, 2) k_basis_r(DevSystem S, DevJob J)
{
    constexpr int NT = 64 * NW, LD = NT + 8, M = 16 * TILES, PS = kRhs * M + 8, LDH = M + 1;
    extern __shared__ __attribute__((aligned(16))) double resident_smem[];
    __shared__ double red[2 * NW];
    __shared__ int s_idx;
    // the right-hand vectors in the order of the dots, P, the partial dots,
    // and per slot the coefficients a, b, a_T, b_T; k; the scalars
    double *SP = resident_smem, *SC = SP + LD, *HP = SC + LD, *Z = HP + LD, *HZ = Z + LD,
           *P = HZ + LD;
    double *part = P + LD, *cf = part + NW * PS, *ck = cf + 4 * M, *scal = ck + M;
    double *Ht = scal + 8, *suj = Ht + M * LDH, *dpart = suj + M;
    short *pinv = reinterpret_cast<short *>(dpart + NW);
    double *T = dpart + NW + NT / 4;
    int *srp = reinterpret_cast<int *>(T + J.q * LD);
    int2 *sblk = reinterpret_cast<int2 *>(srp + ((S.max_nat + 2) & ~1));
    const int nu = J.nu;

    drain_queues(J, &s_idx, [&](int c_, int s_) __attribute__((always_inline)) {
        // values that every lane shares go through v_readfirstlane, so that the
        // control flow on them is scalar
        const int c = uniform(c_), s = uniform(s_);
        // The thread's place passes through an empty asm here and again in every
        // step: otherwise all addresses formed from it are hoisted out of the
        // loops and hold a hundred registers.
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int wv = uniform(tid >> 6), slab = 64 * wv;
        Col g = make_col(S, J, c, O);
        const int n = g.n;
        const int64_t kb0 = S.blk_ptr[g.A];
        const int npat = (int)(S.blk_ptr[g.A + 1] - kb0) * O;
        double *mid = J.mid + (int64_t)s * J.mid_stride;
        double *Up = mid + 2 * (int64_t)nu * nu;
        pinv[tid] = -1;
        // rows past the region stay zero in every vector, so that nothing below
        // asks whether a row exists
        if (tid >= n)
#pragma unroll
            for (int b = 0; b < 6; ++b) SP[b * LD + tid] = 0.0;
        if (tid < 48) SP[(tid >> 3) * LD + NT + (tid & 7)] = 0.0;
        for (int e = tid; e < 8 * J.q; e += NT) T[(e >> 3) * LD + NT + (e & 7)] = 0.0;
        stage_col_index<NT>(S, g, srp, sblk);
        Row<O> w;
        w.k0 = w.k1 = w.ri = 0;
        w.zero = NT / O;
        w.sblk = sblk;
        if (tid < n) {
            const int a = tid / O;
            w.k0 = srp[a];
            w.k1 = srp[a + 1];
            w.ri = tid - a * O;
        }
#pragma unroll
        for (int k = 0; k < Row<O>::KEEP; ++k) {
            const bool in = w.k0 + k < w.k1;
            w.xo[k] = in ? sblk[w.k0 + k].x : w.zero;
        }
        for (int t = tid; t < npat; t += NT) pinv[S.blk_loc[kb0 + t / O] * O + t % O] = (short)t;

        double x;
        int iters, nres, status, start;
        row_cg<O, NW>(S, J, g, w, c, P, red, x, iters, nres, status, start);

        int L = 0;
        if (uniform(status) == 0) {
            double UA[TILES][16], UB[4 * TILES][4];
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int k = 0; k < 16; ++k) UA[t][k] = 0.0;
#pragma unroll
            for (int q = 0; q < 4 * TILES; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) UB[q][r] = 0.0;
            // vector m into its slot; its rows are in LDS at v
            auto insert = [&](int m, const double *v, int l16, int lq) __attribute__((always_inline)) {
                double rows[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) rows[k] = v[slab + 16 * lq + k];
#pragma unroll
                for (int t = 0; t < TILES; ++t)
                    if (t == m / 16)
#pragma unroll
                        for (int k = 0; k < 16; ++k) UA[t][k] = l16 == m % 16 ? rows[k] : UA[t][k];
#pragma unroll
                for (int r = 0; r < 4; ++r) rows[r] = v[slab + 16 * r + l16];
#pragma unroll
                for (int q = 0; q < 4 * TILES; ++q)
                    if (q == m / 4)
#pragma unroll
                        for (int r = 0; r < 4; ++r) UB[q][r] = lq == m % 4 ? rows[r] : UB[q][r];
            };
            bool has_pend = true, b1_live = true, zl = J.q > 0;
            int nb1 = 1, kch = 0, tq = 0, dlast = -1;
            double inv_last = 0.0;
            // The pair's column of vector dlast from the coefficients a, k and the
            // scalars of the step that finished it: four entries per wavefront,
            // one per row of 16 lanes, each a sum over a row of H~.  The diagonal
            // entry needs all of them and follows one step later (dfin).
            int dfin = -1;
            double fin_inv = 0.0, fin_pp = 0.0;
            auto finish_diagonal = [&](int tid) __attribute__((always_inline)) {
                if (dfin >= 0 && tid == 0) {
                    double sd = fin_pp;
                    for (int k = 0; k < NW; ++k) sd -= dpart[k];
                    Ht[dfin * LDH + dfin] = sd * fin_inv * fin_inv;
                }
            };
            auto pair_column = [&](int lane) __attribute__((always_inline)) {
                const int l16 = lane & 15, lq = lane >> 4;
                double dsum = 0.0;
#pragma unroll
                for (int q = 0; q < (M + 4 * NW - 1) / (4 * NW); ++q) {
                    const int m = 4 * (wv + q * NW) + lq;
                    if (4 * (wv + q * NW) >= dlast) continue;
                    double ga = 0.0;
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        const int l = 16 * t + l16;
                        ga += m < dlast && l < dlast ? cf[4 * l] * Ht[m * LDH + l] : 0.0;
                    }
                    ga = sum_within<16>(ga);
                    if (m < dlast && l16 == 0) {
                        const double k = ck[m], gm = k - ga;
                        Ht[m * LDH + dlast] = gm * inv_last;
                        Ht[dlast * LDH + m] = gm * inv_last;
                        dsum += cf[4 * m] * (k + gm);
                    }
                }
                dsum = sum_within<64>(dsum);
                if (lane == 0) dpart[wv] = dsum;
                fin_pp = scal[2];
                if (wv == NW - 1) {
                    // (S u)_j
                    double sj = 0.0;
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        const int l = 16 * t + l16;
                        sj += l < dlast ? cf[4 * l] * suj[l] : 0.0;
                    }
                    sj = (scal[5] - sum_within<16>(sj)) * inv_last;
                    if (lane == 0) {
                        suj[dlast] = sj;
                        Up[nu + dlast] = sj;
                    }
                }
                dfin = dlast;
                fin_inv = inv_last;
            };
            // squared norms of the pending vectors' seeds before any projection
            // (negative: the vector is its own seed)
            double seed_u = -1.0, seed_t = -1.0;
            const int pat = pinv[tid];
            double p = tid == g.jl ? 1.0 : 0.0;   // block 1 starts at e_j
            double z = tid < n ? x : 0.0;         // block 2 at s_j
            P[tid] = p;
            Z[tid] = z;
            for (;;) {
                const int kind = b1_live && nb1 < J.p ? kBlock1 : !zl && tq < kch ? kSeed : kNoCand;
                if (!has_pend && kind == kNoCand && !zl) break;
                int tid = threadIdx.x;
                asm volatile("" : "+v"(tid));
                const int lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
                const bool need_z = zl && kch + 1 < J.q;
                const int pe = J.p + kch, used = zl && pe > L ? pe : L;
                // ---- operator products; the pair's column of the vector finished
                // last while the first blocks' values are on their way ----
                double hm[Row<O>::KEEP][O], sm[Row<O>::KEEP][O];
                load_kept<O>(S.Hd, w, hm);
                load_kept<O>(S.Sd, w, sm);
                __syncthreads();   // staged vectors visible
                if (dlast >= 0) pair_column(lane);
                double hp = 0.0, sp = 0.0, sc = 0.0, hz = 0.0, cand;
                if (kind == kSeed) {
                    const double *seed = T + tq * LD;
                    spmv3<O, true>(S, w, hm, sm, P, seed, hp, sp, sc);
                    cand = seed[tid];
                } else {
                    spmv3<O, false>(S, w, hm, sm, P, Z, hp, sp, hz);
                    cand = hp;
                }
                HP[tid] = hp;
                SP[tid] = sp;
                HZ[tid] = hz;
                if (kind == kBlock1) {
                    __syncthreads();   // H p visible
                    sc = spmv_s<O>(S, w, sm, HP);
                }
                SC[tid] = sc;

                // ---- dots: the basis with S p, S c, H p, the chain with z, H z ----
                wave_sync();
                {
                    const int j = l16 & 3, m0 = (l16 & 12) + lq;
                    double *out = part + wv * PS + j * M + m0;
                    double bv[16];
                    const double *src = SP + (j < 3 ? j : 2) * LD + slab + 16 * lq;
#pragma unroll
                    for (int k = 0; k < 16; ++k) bv[k] = src[k];
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        if (16 * t >= L) continue;
                        double a0 = 0.0, a1 = 0.0;
#pragma unroll
                        for (int k = 0; k < 16; k += 2) {
                            a0 = __builtin_amdgcn_mfma_f64_4x4x4f64(UA[t][k], bv[k], a0, 0, 0, 0);
                            a1 = __builtin_amdgcn_mfma_f64_4x4x4f64(UA[t][k + 1], bv[k + 1], a1, 0, 0, 0);
                        }
                        if (j < 3) out[16 * t] = a0 + a1;
                    }
                    if (zl && kch > 0) {
                        src = Z + (j & 1) * LD + slab + 16 * lq;
#pragma unroll
                        for (int k = 0; k < 16; ++k) bv[k] = src[k];
#pragma unroll
                        for (int t = 0; t < TILES; ++t) {
                            if (16 * t >= pe || 16 * t + 16 <= J.p) continue;
                            double a0 = 0.0, a1 = 0.0;
#pragma unroll
                            for (int k = 0; k < 16; k += 2) {
                                a0 = __builtin_amdgcn_mfma_f64_4x4x4f64(UA[t][k], bv[k], a0, 0, 0, 0);
                                a1 = __builtin_amdgcn_mfma_f64_4x4x4f64(UA[t][k + 1], bv[k + 1], a1, 0, 0, 0);
                            }
                            if (j < 2) out[3 * M + 16 * t] = a0 + a1;
                        }
                    }
                    // pending and chain vector's own dots, (S p)_j, and the
                    // squared norms of the next candidates
                    double v[8] = {p * sp, p * sc, p * hp, z * z, z * hz, tid == g.jl ? sp : 0.0,
                                   cand * sc, hz * hz};
                    lane_reduce8(v);
                    if ((lane & 7) == 0) part[wv * PS + kRhs * M + tr_index<8>(lane)] = v[0];
                }
                __syncthreads();
                finish_diagonal(tid);
                dfin = -1;
                // sums over the wavefronts; zero outside the vectors in use
                for (int e = tid; e < PS; e += NT) {
                    double sum = 0.0;
#pragma unroll
                    for (int k = 0; k < NW; ++k) sum += part[k * PS + e];
                    const int j = e / M, m = e - j * M;
                    const bool in = j < 3 ? m < L : zl && m >= J.p && m < pe;
                    if (j == kRhs) scal[m] = sum;
                    else if (j == 2) ck[m] = in ? sum : 0.0;
                    else cf[4 * m + (j < 2 ? j : j - 1)] = in ? sum : 0.0;
                }
                __syncthreads();

                // ---- decisions (every wavefront; lane l holds the coefficients
                // of slots 16 t + l % 16) ----
                double ca[TILES], cb[TILES], ta[TILES], tb[TILES];
#pragma unroll
                for (int t = 0; t < TILES; ++t) {
                    const double2 ab = *reinterpret_cast<const double2 *>(cf + 4 * (16 * t + l16));
                    const double2 tt = *reinterpret_cast<const double2 *>(cf + 4 * (16 * t + l16) + 2);
                    ca[t] = ab.x;
                    cb[t] = ab.y;
                    ta[t] = tt.x;
                    tb[t] = tt.y;
                }
                bool acc_u = false;
                double f = 0.0, inv_b = 1.0, inv_e = 1.0;
                if (has_pend) {
                    double asq = 0.0, ab = 0.0;
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        asq += ca[t] * ca[t];
                        ab += ca[t] * cb[t];
                    }
                    asq = sum_within<16>(asq);
                    ab = sum_within<16>(ab);
                    const double bb = scal[0] - asq, b0 = seed_u < 0.0 ? bb : seed_u;
                    acc_u = uniform(bb >= DBL_MIN && b0 > 0.0 && !(bb <= J.tau * J.tau * b0));
                    if (acc_u) {
                        inv_b = rsqrt_fast(bb);
                        f = (scal[1] - ab) * inv_b;
                    }
                }
                bool acc_t = false;
                double ft = 0.0;
                if (zl) {
                    double asq = 0.0, ab = 0.0;
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        asq += ta[t] * ta[t];
                        ab += ta[t] * tb[t];
                    }
                    asq = sum_within<16>(asq);
                    ab = sum_within<16>(ab);
                    const double ee = scal[3] - asq, e0 = seed_t < 0.0 ? ee : seed_t;
                    acc_t = uniform(ee >= DBL_MIN && ee > J.tau * J.tau * e0);
                    if (acc_t) {
                        inv_e = rsqrt_fast(ee);
                        ft = (scal[4] - ab) * inv_e;
                    }
                }
                const bool new_pend = (kind == kBlock1 && acc_u) || kind == kSeed;
                const bool new_chain = need_z && acc_t;
                const double scl = kind == kBlock1 ? inv_b : 1.0;

                dlast = acc_u ? L : -1;
                inv_last = inv_b;
                seed_u = scal[6] * scl * scl;
                seed_t = scal[7] * inv_e * inv_e;

                // ---- combinations U a, U b, T a_T, T b_T ----
                double y[4] = {0.0, 0.0, 0.0, 0.0};
                {
                    const double *cq = cf + 4 * lq + (l16 & 3);
#pragma unroll
                    for (int q = 0; q < 4 * TILES; ++q) {
                        if (4 * q >= used) continue;
                        const double a = cq[16 * q];
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            y[r] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, UB[q][r], y[r], 0, 0, 0);
                    }
                }
                transpose4(y);
                // ---- finish u and t, project the candidates once ----
                if (acc_u || new_pend) {
                    const double u = (p - y[0]) * inv_b;
                    p = new_pend ? (cand - y[1] - (acc_u ? f * u : 0.0)) * scl : 0.0;
                    if (acc_u) {
                        if (pat >= 0) Up[(2 + pat) * nu + L] = u;
                        if (tid == g.jl) Up[L] = u;
                        SP[tid] = u;
                    }
                } else {
                    p = 0.0;
                }
                P[tid] = p;
                if (acc_t) {
                    const double t = (z - y[2]) * inv_e;
                    z = new_chain ? (hz - y[3] - ft * t) * inv_e : 0.0;
                    Z[tid] = z;
                    T[kch * LD + tid] = t;
                }
                // the finished vectors into their slots (the wavefront's own rows)
                wave_sync();
                if (acc_u) insert(L, SP, l16, lq);
                if (acc_t) insert(pe, T + kch * LD, l16, lq);
                if (kind == kBlock1) {
                    if (acc_u) ++nb1;
                    else b1_live = false;
                }
                if (kind == kSeed) ++tq;
                if (zl) {
                    if (acc_t) ++kch;
                    zl = new_chain;
                }
                if (acc_u) ++L;
                has_pend = new_pend;
            }
            __syncthreads();
            if (dlast >= 0) pair_column(tid & 63);
            __syncthreads();
            finish_diagonal(tid);
            __syncthreads();   // H~ visible
            for (int e = tid; e < L * L; e += NT) {
                const int m = e / L, k = e - m * L;
                mid[m * nu + k] = Ht[m * LDH + k];
                mid[nu * nu + m * nu + k] = m == k ? 1.0 : 0.0;
            }
        }
        if (tid == 0) write_stats(J, c, L, iters, nres, status, start);
        __syncthreads();
    });
}

// A shape: regions of at most `rows` orbitals, at most `vecs` vectors.
struct Shape {
    int rows, vecs;
    int64_t (*doubles)(int q);
    void *k4;
};

template <int NW, int TILES>
Shape shape()
{
    return {64 * NW, 16 * TILES, resident_doubles<NW, TILES>, (void *)k_basis_r<4, NW, TILES>};
}

const Shape *pick(int o, int nmax, int nu, int q, size_t index_bytes)
{
    static const Shape shapes[] = {shape<4, 1>(), shape<4, 2>(), shape<8, 2>()};
    if (o != 4) return nullptr;
    for (const Shape &s : shapes)
        if (nmax <= s.rows && nu <= s.vecs &&
            sizeof(double) * (size_t)s.doubles(q) + index_bytes <= 159 * 1024)
            return &s;
    return nullptr;
}

}  // namespace

bool basis_resident_fits(int nmax, int nu, int q, int o, int precision, size_t index_bytes)
{
    return precision == 0 && pick(o, nmax, nu, q, index_bytes) != nullptr;
}

void *basis_r_kernel(int o, int nmax, int nu, int q, size_t index_bytes, int *threads, size_t *smem)
{
    const Shape *s = pick(o, nmax, nu, q, index_bytes);
    if (!s) return nullptr;
    *threads = s->rows;
    *smem = sizeof(double) * (size_t)s->doubles(q) + index_bytes;
    return s->k4;
}

}  // namespace ma
