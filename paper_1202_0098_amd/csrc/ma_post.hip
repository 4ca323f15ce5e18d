// Quantities built from the column outputs of a solve (gfx950):
//
//   forces   F_K = -spin sum_j sum_i [rho_ij dH_ji/dR_K - pi_ij dS_ji/dR_K]
//            (Sec. 2: the force as a sum of partial sums over the columns j;
//            only pattern elements enter, and the derivative blocks are
//            nonzero only between neighbouring atoms)
//   DOS      D(E) = spin/pi sum_j sum_a w_a eta / ((E - eps_a)^2 + eta^2),
//            the S-weighted trace of the subspace Green's functions at
//            E + i eta (Eqs. 11-12), from the Ritz values and weights
//   G(z)     G_ij(z) = sum_a v_ia v_ja / (z - eps_a) at the pattern
//            elements (Eq. 12 applied to e_j, Eq. 11), from the stored
//            amplitudes v_ia v_ja of a solve that bisected mu
//
// All reductions run in a fixed order: results are bitwise reproducible.
#include "ma_device.h"

namespace ma {

namespace {

// F_X = spin sum over blocks k = (X, B), B != X, of g_k - g_T(k), where
// g_k = sum_{r,c} rho_k[r][c] dH_k[:][r][c] - pi_k[r][c] dS_k[:][r][c] and
// T(k) is the block (B, X).  Block k = (A, B) holds columns j = (A, r) at
// rows i = (B, c); dH_k is the derivative of H_AB with respect to R_B, so
// g_k enters F_A with + and F_B with -.
//
// The g of an atom nearly cancel, so that their own rounding would be most of the
// result's error: sums carry what their additions round off (Knuth's two-sum) to
// the end.  Not a number there where the sum itself is not finite; such a sum is
// taken as it is.
struct Sum2 {
    double h = 0.0, l = 0.0;
    __device__ __forceinline__ void add(double v)
    {
        const double s = h + v, w = s - h;
        l += (h - (s - w)) + (v - w);
        h = s;
    }
    __device__ __forceinline__ void add(const Sum2 &v)
    {
        add(v.h);
        l += v.l;
    }
    __device__ __forceinline__ double value() const { return isfinite(h) ? h + l : h; }
};

template <int CTRL>
__device__ __forceinline__ void add_dpp(Sum2 &s, const Sum2 &from)
{
    Sum2 o;
    o.h = dpp<CTRL>(from.h);
    o.l = dpp<CTRL>(from.l);
    s.add(o);
}

// Exchange steps of a transposed reduction: a's sum in one half of the lanes,
// b's in the other (where `other` holds).
__device__ __forceinline__ void fold32(Sum2 &a, Sum2 b)
{
    swap32(a.h, b.h);
    swap32(a.l, b.l);
    a.add(b);
}

__device__ __forceinline__ void fold16(Sum2 &a, Sum2 b)
{
    swap16(a.h, b.h);
    swap16(a.l, b.l);
    a.add(b);
}

template <int CTRL>
__device__ __forceinline__ void fold_dpp(Sum2 &a, const Sum2 &b, bool other)
{
    Sum2 send;
    send.h = other ? a.h : b.h;
    send.l = other ? a.l : b.l;
    a.h = other ? b.h : a.h;
    a.l = other ? b.l : a.l;
    add_dpp<CTRL>(a, send);
}

// Sums over each group of W lanes (4, 16 or 64) of three values per lane; value v's
// ends in s[0] of the group's lane first_lane<W>(v).
template <int W>
__device__ __forceinline__ int first_lane(int v)
{
    return v == 0 ? 0 : W == 64 ? (v == 1 ? 16 : 32) : W == 16 ? (v == 1 ? 8 : 4) : (v == 1 ? 2 : 1);
}

template <int W>
__device__ __forceinline__ void group_sums(Sum2 (&s)[3])
{
    const int l = threadIdx.x;
    if constexpr (W == 64) {
        fold32(s[0], s[2]);
        fold32(s[1], Sum2());
        fold16(s[0], s[1]);
        add_dpp<kDppRor8>(s[0], s[0]);
        add_dpp<kDppHalfMirror>(s[0], s[0]);
        add_dpp<kDppXor2>(s[0], s[0]);
        add_dpp<kDppXor1>(s[0], s[0]);
    } else if constexpr (W == 16) {
        fold_dpp<kDppRor8>(s[0], s[1], (l & 8) != 0);
        add_dpp<kDppRor8>(s[2], s[2]);
        fold_dpp<kDppHalfMirror>(s[0], s[2], (l & 4) != 0);
        add_dpp<kDppXor2>(s[0], s[0]);
        add_dpp<kDppXor1>(s[0], s[0]);
    } else {
        fold_dpp<kDppXor2>(s[0], s[1], (l & 2) != 0);
        add_dpp<kDppXor2>(s[2], s[2]);
        fold_dpp<kDppXor1>(s[0], s[2], (l & 1) != 0);
    }
}

// In one launch: one wavefront per atom, LPB lanes per block.  It reads every block
// twice (as k and as T(k)), which costs less than a second launch while the blocks
// are few and small; also where there is no memory for the block sums.
template <int LPB>
__global__ void __launch_bounds__(64) k_forces_direct(int n_atoms, int oo, const int64_t *blk_ptr,
                                                      const int32_t *blk_col, const int32_t *blk_t,
                                                      const double *dH, const double *dS,
                                                      const double *rho, const double *pi,
                                                      double spin, double *F)
{
    const int lane = threadIdx.x;
    for (int X = blockIdx.x; X < n_atoms; X += gridDim.x) {
        Sum2 f[3];
        for (int64_t k = blk_ptr[X] + lane / LPB; k < blk_ptr[X + 1]; k += 64 / LPB) {
            if (blk_col[k] == X) continue;
            const int64_t kt = blk_t[k];
            for (int e = lane % LPB; e < oo; e += LPB) {
                const double ra = rho[k * oo + e], pa = pi[k * oo + e];
                const double rb = rho[kt * oo + e], pb = pi[kt * oo + e];
                const double *ha = dH + k * 3 * oo + e, *sa = dS + k * 3 * oo + e;
                const double *hb = dH + kt * 3 * oo + e, *sb = dS + kt * 3 * oo + e;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    f[d].add(ra * ha[d * oo] - pa * sa[d * oo]);
                    f[d].add(pb * sb[d * oo] - rb * hb[d * oo]);
                }
            }
        }
        group_sums<64>(f);
#pragma unroll
        for (int d = 0; d < 3; ++d)
            if (lane == first_lane<64>(d)) F[3 * (int64_t)X + d] = spin * f[0].value();
    }
}

// Otherwise g_k first, which reads every value once: sums and carries, six doubles
// per block, LPB lanes per block (a quarter of the lanes, with fewer lines of memory
// in flight: 1.4 times the time).  Bound by the bytes (64 o^2 per block): 2,048 spd
// atoms 67 us and 4 us for the sums below, where one wavefront per atom with the
// blocks and their transposes took 122; error in the 2-norm 4.9e-17 of the
// forces, with plain sums 2.3e-16, by one wavefront per atom 1.2e-16.
template <int LPB>
__global__ void __launch_bounds__(256) k_block_forces(int64_t nblk, int oo, const double *dH,
                                                      const double *dS, const double *rho,
                                                      const double *pi, double *g)
{
    constexpr int BPW = 256 / LPB;   // blocks per workgroup
    const int l = threadIdx.x % LPB;
    for (int64_t k = (int64_t)blockIdx.x * BPW + threadIdx.x / LPB; k - threadIdx.x / LPB < nblk;
         k += (int64_t)gridDim.x * BPW) {
        Sum2 f[3];
        if (k < nblk && l < oo) {
            // (the first terms need no additions)
            auto term = [&](int e, int d) __attribute__((always_inline)) {
                const int64_t at = (k * 3 + d) * oo + e;
                return rho[k * oo + e] * dH[at] - pi[k * oo + e] * dS[at];
            };
#pragma unroll
            for (int d = 0; d < 3; ++d) f[d].h = term(l, d);
#pragma unroll 2
            for (int e = l + LPB; e < oo; e += LPB)
#pragma unroll
                for (int d = 0; d < 3; ++d) f[d].add(term(e, d));
        }
        group_sums<LPB>(f);
        if (k < nblk)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if (l == first_lane<LPB>(d)) {
                    g[6 * k + d] = f[0].h;
                    g[6 * k + 3 + d] = f[0].l;
                }
    }
}

// Then the sum over an atom's blocks, LPA lanes per atom.
template <int LPA>
__global__ void __launch_bounds__(256) k_forces(int n_atoms, const int64_t *blk_ptr,
                                                const int32_t *blk_col, const int32_t *blk_t,
                                                const double *g, double spin, double *F)
{
    constexpr int APW = 256 / LPA;   // atoms per workgroup
    const int l = threadIdx.x % LPA, sub = threadIdx.x / LPA;
    for (int X0 = blockIdx.x * APW; X0 < n_atoms; X0 += gridDim.x * APW) {
        const int X = X0 + sub;
        Sum2 f[3];
        if (X < n_atoms)
            for (int64_t k = blk_ptr[X] + l; k < blk_ptr[X + 1]; k += LPA) {
                if (blk_col[k] == X) continue;
                const double *a = g + 6 * k, *b = g + 6 * (int64_t)blk_t[k];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    f[d].add(a[d]);
                    f[d].add(-b[d]);
                    f[d].l += a[3 + d] - b[3 + d];
                }
            }
        group_sums<LPA>(f);
        if (X < n_atoms)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if (l == first_lane<LPA>(d)) F[3 * (int64_t)X + d] = spin * f[0].value();
    }
}

constexpr int kDosStage = 1024;   // Ritz pairs staged at a time by the DOS kernel
static_assert(kDosChunkMax % kDosStage == 0, "whole stages");
constexpr int kDosTile = 512;     // energies per workgroup, two per thread

}  // namespace

// Ritz pairs per workgroup: stages of 1,024 until the launch has 2,048
// workgroups, at most eight (which bounds the partial sums)
int64_t dos_chunk(int ncols, int nu, int nE)
{
    const int64_t npairs = (int64_t)ncols * nu;
    const int64_t wgs = (npairs + kDosStage - 1) / kDosStage * ((nE + kDosTile - 1) / kDosTile);
    return std::max<int64_t>(kDosStage, std::min<int64_t>(kDosChunkMax, wgs / 2048 * kDosStage));
}

namespace {

// Partial DOS of one chunk of Ritz pairs (staged in LDS) at a tile of
// energies: part[chunk][E] (thread t takes energies tile * 512 + t and + 256).
// Bound by the evaluations: the reciprocal is v_rcp_f64 with one third-order
// correction (within 1 ulp).  491,520 pairs at 500 energies 92 us; with IEEE
// divisions and 8,192 pairs per workgroup, which left half of the compute units
// idle, 390 us.
__global__ void __launch_bounds__(256) k_dos_part(const double *eps, const double *wts,
                                                  const int32_t *stats, int ncols, int nu,
                                                  int64_t chunk, const double *E, int nE,
                                                  double eta, double *part)
{
    __shared__ double2 pair[kDosStage];
    const int64_t npairs = (int64_t)ncols * nu;
    const int64_t p0 = (int64_t)blockIdx.x * chunk;
    const int i0 = blockIdx.y * kDosTile + threadIdx.x, i1 = i0 + 256;
    const double e0 = i0 < nE ? E[i0] : 0.0, e1 = i1 < nE ? E[i1] : 0.0;
    const double eta2 = eta * eta;
    // where a denominator may leave the range of the fast reciprocal (or a value
    // is not finite) the workgroup divides
    const bool far = !(fabs(e0) < 1e100) || !(fabs(e1) < 1e100) || !(eta2 > 1e-200 && eta2 < 1e200);
    double a0 = 0.0, a1 = 0.0;
    for (int64_t s0 = p0; s0 < p0 + chunk && s0 < npairs; s0 += kDosStage) {
        const int cnt = (int)min<int64_t>(kDosStage, npairs - s0);
        bool plain = far;
        __syncthreads();
        for (int t = threadIdx.x; t < cnt; t += 256) {
            const int64_t g = s0 + t;
            const int c = (int)(g / nu), a = (int)(g - (int64_t)c * nu);
            const bool ok = a < stats[(int64_t)c * kStats];
            const double ep = ok ? eps[g] : 0.0;
            pair[t] = make_double2(ep, ok ? wts[g] * eta : 0.0);
            plain = plain || !(fabs(ep) < 1e100);
        }
        if (__syncthreads_or(plain)) {
            for (int t = 0; t < cnt; ++t) {
                const double2 q = pair[t];
                const double d0 = e0 - q.x, d1 = e1 - q.x;
                a0 += q.y / (d0 * d0 + eta2);
                a1 += q.y / (d1 * d1 + eta2);
            }
            continue;
        }
#pragma unroll 4
        for (int t = 0; t < cnt; ++t) {
            const double2 q = pair[t];
            const double d0 = e0 - q.x, d1 = e1 - q.x;
            const double x0 = fma(d0, d0, eta2), x1 = fma(d1, d1, eta2);
            const double y0 = __builtin_amdgcn_rcp(x0), y1 = __builtin_amdgcn_rcp(x1);
            const double r0 = fma(-x0, y0, 1.0), r1 = fma(-x1, y1, 1.0);
            a0 = fma(q.y, fma(y0, fma(r0, r0, r0), y0), a0);
            a1 = fma(q.y, fma(y1, fma(r1, r1, r1), y1), a1);
        }
    }
    if (i0 < nE) part[(int64_t)blockIdx.x * nE + i0] = a0;
    if (i1 < nE) part[(int64_t)blockIdx.x * nE + i1] = a1;
}

// D(E) = spin / pi * sum over chunks: 16 energies per workgroup, thread (group,
// energy) takes chunks group, group + 16, ...; the groups are added in order
__global__ void __launch_bounds__(256) k_dos_sum(const double *part, int nchunks, int nE,
                                                 double spin, double *out)
{
    __shared__ double red[16][17];
    const int v = threadIdx.x & 15, u = threadIdx.x >> 4;
    const int ie = blockIdx.x * 16 + v;
    double s = 0.0;
    if (ie < nE) {
#pragma unroll 8
        for (int c = u; c < nchunks; c += 16) s += part[(int64_t)c * nE + ie];
    }
    red[u][v] = s;
    __syncthreads();
    if (u == 0 && ie < nE) {
        s = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) s += red[k][v];
        out[ie] = spin / M_PI * s;
    }
}

// G_ij(z) at the pattern slots of every solved column from the stored
// amplitudes (TA: FP64 or FP32), one workgroup per column.
template <typename TA>
__global__ void __launch_bounds__(128) k_green(DevSystem S, DevJob J, double zr, double zi,
                                               double *gre, double *gim)
{
    __shared__ double cr[kMaxNu], ci[kMaxNu];
    const int o = S.o, nu = J.nu;
    for (int c = blockIdx.x; c < J.ncols; c += gridDim.x) {
        const int j = J.cols[c];
        const int A = j / o, r = j - A * o;
        const int L = J.stats[(int64_t)c * kStats];
        __syncthreads();
        for (int a = threadIdx.x; a < nu; a += blockDim.x) {
            // 1 / (z - eps) = conj(z - eps) / |z - eps|^2
            const double dr = zr - J.eps[(int64_t)c * nu + a], di = zi;
            const double den = dr * dr + di * di;
            cr[a] = a < L ? dr / den : 0.0;
            ci[a] = a < L ? -di / den : 0.0;
        }
        __syncthreads();
        const int64_t kb0 = S.blk_ptr[A];
        const int npat = (int)(S.blk_ptr[A + 1] - kb0) * o;
        const TA *amp = reinterpret_cast<const TA *>(J.amp) + J.amp_off[c];
        for (int t = threadIdx.x; t < npat; t += blockDim.x) {
            double sr = 0.0, si = 0.0;
            for (int a = 0; a < L; ++a) {
                const double am = (double)amp[t * nu + a];
                sr += cr[a] * am;
                si += ci[a] * am;
            }
            const int64_t slot = ((kb0 + t / o) * o + r) * o + (t % o);
            if (gre) gre[slot] = sr;
            if (gim) gim[slot] = si;
        }
    }
}

// Start vectors from kept s_j: for column c (global j, atom A), row i of
// the current region of A (atom b = its i / o-th atom) takes the kept value
// of the same orbital of b in A's region at the time of keeping, or zero if b
// was not in it (both atom lists ascending: binary search).
__global__ void __launch_bounds__(128) k_map_sj(int ncols, const int32_t *cols, int o,
                                                RegionView cur, RegionView old,
                                                const double *store, const int32_t *have,
                                                double *x0full)
{
    for (int c = blockIdx.x; c < ncols; c += gridDim.x) {
        const int j = cols[c];
        const int A = j / o;
        const int rid = cur.reg_id[A], orid = old.reg_id[A];
        const int32_t *ca = cur.reg_atoms + cur.reg_off[rid];
        const int32_t *oa = old.reg_atoms + old.reg_off[orid];
        const int len = cur.reg_len[rid], olen = old.reg_len[orid];
        const bool kept = have[j] != 0;
        const double *src = store + (int64_t)j * old.nmax;
        double *dst = x0full + (int64_t)c * cur.nmax;
        for (int t = threadIdx.x; t < len; t += blockDim.x) {
            const int b = ca[t];
            int lo = 0, hi = olen;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (oa[mid] < b) lo = mid + 1;
                else hi = mid;
            }
            const bool found = kept && lo < olen && oa[lo] == b;
            for (int r = 0; r < o; ++r) dst[t * o + r] = found ? src[lo * o + r] : 0.0;
        }
    }
}

}  // namespace

hipError_t launch_map_sj(int ncols, const int32_t *cols, int o, RegionView cur, RegionView old,
                         const double *store, const int32_t *have, double *x0full, hipStream_t st)
{
    const int grid = ncols < 65536 ? ncols : 65536;
    hipLaunchKernelGGL(k_map_sj, dim3(grid), dim3(128), 0, st, ncols, cols, o, cur, old, store,
                       have, x0full);
    return hipGetLastError();
}

// Up to 16 values per block (o <= 4) and 16,384 blocks one launch (fastest call of
// 3,000, with its synchronisation: 1,000 sp3 atoms 22.0 us, in two launches 24.3; 2,744
// atoms, 13,720 blocks, 24.6 either way; 4,096 atoms 26.1 and 24.9).
bool forces_need_blocks(int o, int64_t nblk) { return o > 4 || nblk > 16384; }

hipError_t launch_forces(int n_atoms, int o, const int64_t *blk_ptr, const int32_t *blk_col,
                         const int32_t *blk_t, const double *dH, const double *dS,
                         const double *rho, const double *pi, double spin, int64_t nblk,
                         double *g, double *F, hipStream_t st)
{
    const int oo = o * o;
    auto grid = [](int64_t n) { return dim3((unsigned)(n < (1 << 20) ? n : (1 << 20))); };
    if (!g) {
        hipLaunchKernelGGL(oo <= 16 ? k_forces_direct<16> : k_forces_direct<64>, grid(n_atoms), dim3(64), 0,
                           st, n_atoms, oo, blk_ptr, blk_col, blk_t, dH, dS, rho, pi, spin, F);
        return hipGetLastError();
    }
    if (oo <= 16)
        hipLaunchKernelGGL(k_block_forces<16>, grid((nblk + 15) / 16), dim3(256), 0, st, nblk, oo, dH, dS,
                           rho, pi, g);
    else
        hipLaunchKernelGGL(k_block_forces<64>, grid((nblk + 3) / 4), dim3(256), 0, st, nblk, oo, dH, dS,
                           rho, pi, g);
    if (nblk <= 16 * (int64_t)n_atoms)
        hipLaunchKernelGGL(k_forces<16>, grid((n_atoms + 15) / 16), dim3(256), 0, st, n_atoms, blk_ptr,
                           blk_col, blk_t, g, spin, F);
    else
        hipLaunchKernelGGL(k_forces<64>, grid((n_atoms + 3) / 4), dim3(256), 0, st, n_atoms, blk_ptr,
                           blk_col, blk_t, g, spin, F);
    return hipGetLastError();
}

size_t dos_partial_doubles(int ncols, int nu, int nE, int64_t chunk)
{
    const int64_t npairs = (int64_t)ncols * nu;
    return (size_t)((npairs + chunk - 1) / chunk) * nE;
}

hipError_t launch_dos(const double *eps, const double *wts, const int32_t *stats, int ncols,
                      int nu, const double *E, int nE, double eta, double spin, int64_t chunk,
                      double *part, double *out, hipStream_t st)
{
    const int64_t npairs = (int64_t)ncols * nu;
    const int nchunks = (int)((npairs + chunk - 1) / chunk);
    const int tiles = (nE + kDosTile - 1) / kDosTile;
    if (nchunks < 1 || tiles < 1) return hipSuccess;
    hipLaunchKernelGGL(k_dos_part, dim3(nchunks, tiles), dim3(256), 0, st, eps, wts, stats, ncols,
                       nu, chunk, E, nE, eta, part);
    hipLaunchKernelGGL(k_dos_sum, dim3((nE + 15) / 16), dim3(256), 0, st, part, nchunks, nE, spin, out);
    return hipGetLastError();
}

hipError_t launch_green(const DevSystem &S, const DevJob &J, double zr, double zi, double *gre,
                        double *gim, hipStream_t st)
{
    const int grid = J.ncols < 65536 ? J.ncols : 65536;
    if (J.precision == 0)
        hipLaunchKernelGGL(k_green<double>, dim3(grid), dim3(128), 0, st, S, J, zr, zi, gre, gim);
    else
        hipLaunchKernelGGL(k_green<float>, dim3(grid), dim3(128), 0, st, S, J, zr, zi, gre, gim);
    return hipGetLastError();
}

}  // namespace ma
