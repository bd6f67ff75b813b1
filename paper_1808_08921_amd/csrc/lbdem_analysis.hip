// lbdem_analysis.hip -- dispersion analysis of probe records (Sec. 3.2).
//
// Space-time DFT of a probe record x[t][z] on a chosen (omega, kappa) grid, the ridge of its
// spectrum, and the fit of the stationary lossy wave of Eq. (1Dwave).  FP64 throughout.
//
// The record is real, so a segment of rows is folded about its centre tc, S = x(tc + tau) +
// x(tc - tau), D = x(tc + tau) - x(tc - tau), tau = 1/2, 3/2, ..., and
//   sum x(t) exp(-j omega t) = exp(-j omega tc) (sum S cos(omega tau) - j sum D sin(omega tau)),
// half the multiplications of the unfolded sum.  The two sums over tau are products of a
// (frequency x tau) and a (tau x column) matrix and run on the matrix units in FP64.  Time is
// split over waves and chunks whose partial sums are added in a fixed order (deterministic), then
// the space stage multiplies by a table of exp(j kappa_n z).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <mutex>
#include <stdint.h>

#include "lbdem_internal.hpp"

namespace lbdem {

namespace {

constexpr int kAnchor = 64;   // rotations between exact phases
constexpr int kMT = 2;        // tiles of 16 frequencies per wave in the time stage
constexpr int kCus = 256;
constexpr int kTimeBlocks = 2 * kCus; // two workgroups a CU
constexpr long long kSplitRow = 131072; // elements of E a row reads from which it is split

typedef double d4 __attribute__((ext_vector_type(4)));

// Maximum and minimum over the 64 lanes in vector instructions (rows of 16 lanes, then the
// rows); no lane holds a NaN
template <int CTRL> __device__ inline int dpp(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false); }
template <int CTRL> __device__ inline double dpp(double v)
{
    return __hiloint2double(dpp<CTRL>(__double2hiint(v)), dpp<CTRL>(__double2loint(v)));
}
__device__ inline double lane_of(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ inline double wave_max(double v)
{
    v = fmax(v, dpp<0xB1>(v));  // quad_perm [1,0,3,2]
    v = fmax(v, dpp<0x4E>(v));  // quad_perm [2,3,0,1]
    v = fmax(v, dpp<0x141>(v)); // row_half_mirror
    v = fmax(v, dpp<0x140>(v)); // row_mirror
    return fmax(fmax(lane_of(v, 0), lane_of(v, 16)), fmax(lane_of(v, 32), lane_of(v, 48)));
}
__device__ inline int wave_min(int v)
{
    v = min(v, dpp<0xB1>(v));
    v = min(v, dpp<0x4E>(v));
    v = min(v, dpp<0x141>(v));
    v = min(v, dpp<0x140>(v));
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

__device__ inline double2 cmul_acc(double2 acc, double2 a, double2 b)
{
    // acc + a * b (complex)
    acc.x = fma(a.x, b.x, fma(-a.y, b.y, acc.x));
    acc.y = fma(a.x, b.y, fma(a.y, b.x, acc.y));
    return acc;
}

// One wave per 16 kMT frequencies, 16 NT columns and `seg` rows; the four waves of a workgroup
// take four segments of a chunk.  Operands of the 16 x 16 x 4 products (lane l: frequency or
// column l % 16, tau index l / 16): the phases are advanced by a rotation per four tau in
// registers and set exactly every kAnchor rotations; the record is read straight into the lanes
// that need it, kAhead steps ahead.  Bound by the matrix units (20000 rows x 24 columns x 1024
// frequencies: 18 us at the rate of a large FP64 matrix product, with the columns' padding to 32;
// 37 us, the matrix units busy in 45 % of the cycles; 64 us for the unfolded sum on the vector
// units, which waited for its broadcasts from LDS.  kMT = 4 or one workgroup a CU: 37 us as well).
template <int NT>
__global__ __launch_bounds__(256, 2) void k_dft_time(const double *__restrict__ x, long long nt, int nz, double t0,
                                                     double w0, double dw, int nw, int nwb, long long seg,
                                                     double2 *__restrict__ part)
{
    constexpr int kAhead = 4;
    __shared__ d4 red[2][2 * kMT * NT][64];
    __shared__ double2 anchor[4][16 * kMT];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i16 = lane & 15, kq = lane >> 4;
    const int m0 = (int)(blockIdx.x % nwb) * 16 * kMT;
    const long long c = blockIdx.x / nwb;
    const int z0 = blockIdx.y * 16 * NT;
    const long long ta = min((c * 4 + __builtin_amdgcn_readfirstlane(wv)) * seg, nt), tb = min(ta + seg, nt);
    // rows tc + 1/2 + h and tc - 1/2 - h, h = kq + 4 k (a segment has fewer than 2^30 rows)
    const int n = (int)(tb - ta), hs = (n + 1) / 2, nstep = (hs + 3) / 4;
    const double tc = (double)(ta + hs) - 0.5;
    const double *xs = x + ta * nz;
    double om[kMT], co[kMT], si[kMT], rc[kMT], rs[kMT];
#pragma unroll
    for (int f = 0; f < kMT; ++f) {
        om[f] = w0 + (double)(m0 + 16 * f + i16) * dw;
        sincos(om[f] * 4.0, &rs[f], &rc[f]);
    }
    d4 re[kMT][NT], im[kMT][NT]; // sum S cos, sum D sin
#pragma unroll
    for (int f = 0; f < kMT; ++f)
#pragma unroll
        for (int q = 0; q < NT; ++q) re[f][q] = im[f][q] = (d4){0.0, 0.0, 0.0, 0.0};
    double up[kAhead][NT], lo[kAhead][NT];
    // (a step past the segment repeats its last one, a row past it the nearest one, and is left
    // out when it is used; a column past the record repeats its last one and is not stored.
    // Row bases in scalar registers, 32-bit offsets of at most three rows per lane)
    auto fetch = [&](int k, int slot) {
        const int h0 = 4 * min(k, nstep - 1), ra = min(hs + h0, n - 1);
        const int more = min(n - 1 - ra, 3), less = min(hs - 1 - h0, 3);
        const char *a = (const char *)(xs + (long long)ra * nz);
        const char *b = (const char *)(xs + (long long)(hs - 1 - h0 - less) * nz);
        const unsigned oa = __umul24(min(kq, more), nz), ob = __umul24(less - min(kq, less), nz);
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const unsigned z = (unsigned)min(z0 + 16 * q + i16, nz - 1);
            up[slot][q] = *(const double *)(a + (oa + z) * 8u);
            lo[slot][q] = *(const double *)(b + (ob + z) * 8u);
        }
        // (otherwise the compiler makes one load of those before and in the loop, at the loop's
        // head, where it is waited for)
        asm volatile("" ::: "memory");
    };
    if (nstep > 0)
#pragma unroll
        for (int k = 0; k < kAhead; ++k) fetch(k, k);
    for (int k0 = 0; k0 < nstep; k0 += kAhead) {
        if (k0 % kAnchor == 0)
#pragma unroll
            for (int f = 0; f < kMT; ++f) sincos(om[f] * ((double)(4 * k0 + kq) + 0.5), &si[f], &co[f]);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const int h = kq + 4 * (k0 + j);
            const bool has_a = hs + h < n, has_b = h < hs;
            double S[NT], D[NT];
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                const double va = has_a ? up[j][q] : 0.0, vb = has_b ? lo[j][q] : 0.0;
                S[q] = va + vb;
                D[q] = va - vb;
            }
            fetch(k0 + j + kAhead, j);
#pragma unroll
            for (int f = 0; f < kMT; ++f) {
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    re[f][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(co[f], S[q], re[f][q], 0, 0, 0);
                    im[f][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(si[f], D[q], im[f][q], 0, 0, 0);
                }
                const double cn = fma(co[f], rc[f], -si[f] * rs[f]);
                si[f] = fma(si[f], rc[f], co[f] * rs[f]);
                co[f] = cn;
            }
        }
    }
    // exp(-j omega (t0 + tc)) (re - j im); a product's element r of lane l is frequency l / 16 + 4 r
    // (one frequency's factor per lane, through LDS)
    {
        double a_s, a_c;
        sincos((w0 + (double)(m0 + (lane & (16 * kMT - 1))) * dw) * (t0 + tc), &a_s, &a_c);
        if (lane < 16 * kMT) anchor[wv][lane] = make_double2(a_c, a_s);
    }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < kMT; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double2 a = anchor[wv][16 * f + kq + 4 * r];
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                const double p = re[f][q][r], d = im[f][q][r];
                re[f][q][r] = fma(a.x, p, -a.y * d);
                im[f][q][r] = fma(-a.x, d, -a.y * p);
            }
        }
    // the four segments: (0 + 2) + (1 + 3)
    for (int half = 2; half >= 1; half >>= 1) {
        __syncthreads();
        if (wv >= half && wv < 2 * half)
#pragma unroll
            for (int f = 0; f < kMT; ++f)
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    red[wv - half][2 * (f * NT + q)][lane] = re[f][q];
                    red[wv - half][2 * (f * NT + q) + 1][lane] = im[f][q];
                }
        __syncthreads();
        if (wv < half)
#pragma unroll
            for (int f = 0; f < kMT; ++f)
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    re[f][q] += red[wv][2 * (f * NT + q)][lane];
                    im[f][q] += red[wv][2 * (f * NT + q) + 1][lane];
                }
    }
    if (wv != 0) return;
#pragma unroll
    for (int f = 0; f < kMT; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + 16 * f + kq + 4 * r;
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                const int z = z0 + 16 * q + i16;
                if (m < nw && z < nz) part[((size_t)c * nw + m) * nz + z] = make_double2(re[f][q][r], im[f][q][r]);
            }
        }
}

// The first sum_blocks workgroups: G[m][z] = sum over chunks, in chunk order; the others:
// E[z][n] = exp(j kappa_n zpos[z])
__global__ __launch_bounds__(256) void k_dft_sum(const double2 *__restrict__ part, long long nmz, int nchunk,
                                                 double2 *__restrict__ G, unsigned sum_blocks,
                                                 const double *__restrict__ zpos, int nz, double k0, double dk, int nk,
                                                 double2 *__restrict__ E)
{
    if (blockIdx.x < sum_blocks) {
        const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
        if (i >= nmz) return;
        double2 a = part[i];
#pragma unroll 8
        for (int c = 1; c < nchunk; ++c) {
            const double2 b = part[(size_t)c * nmz + i];
            a.x += b.x;
            a.y += b.y;
        }
        G[i] = a;
        return;
    }
    const long long i = (long long)(blockIdx.x - sum_blocks) * 256 + threadIdx.x;
    if (i >= (long long)nz * nk) return;
    const int z = (int)(i / nk), n = (int)(i % nk);
    const double ka = k0 + (double)n * dk;
    double s, c;
    sincos(ka * zpos[z], &s, &c);
    E[i] = make_double2(c, s);
}

// ridge[m0 + r], the first n of the largest |F|^2 in row m0 + r (-1 if none compares), from each
// thread's largest and its n
template <int MR>
__device__ inline void store_ridge(const double (&best)[MR], const int (&first)[MR], int m0, int nw,
                                   int *__restrict__ ridge)
{
    __shared__ double s_p[16][MR];
    __shared__ int s_n[16][MR];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
#pragma unroll
    for (int r = 0; r < MR; ++r) {
        const double top = wave_max(best[r]);
        const int n = wave_min(best[r] == top ? first[r] : 0x7fffffff);
        if (lane == 0) {
            s_p[wv][r] = top;
            s_n[wv][r] = n;
        }
    }
    __syncthreads();
    if (threadIdx.x < MR && m0 + (int)threadIdx.x < nw) {
        double b = s_p[0][threadIdx.x];
        int n = s_n[0][threadIdx.x];
        for (int w = 1; w < nwv; ++w) {
            const double ob = s_p[w][threadIdx.x];
            const int on = s_n[w][threadIdx.x];
            if (ob > b || (ob == b && on < n)) {
                b = ob;
                n = on;
            }
        }
        ridge[m0 + threadIdx.x] = n == 0x7fffffff ? -1 : n;
    }
}

// F[m][n] = sum_z G[m][z] E[z][n] for MR rows m and the n of this workgroup (all of them, or one
// of `parts` parts), and with ridge the rows' ridge, for which the workgroup has to hold every n.
// (Workgroups of neighbouring numbers take the parts of the same rows: with a multiple of 8 of
// them each XCD keeps to its parts of E, which then stay in its L2.)  An element of E serves MR
// rows, and a row's maximum needs no second pass over F (1024 x 1024 x 24: 17 + 7 us one row and
// 256 n at a time with a kernel for the ridge, 12 us).  UZ: loads in flight.
template <int MR, int UZ>
__global__ __launch_bounds__(1024) void k_dft_space(const double2 *__restrict__ G, const double2 *__restrict__ E,
                                                    int nz, int nw, int nk, double2 *__restrict__ F,
                                                    int *__restrict__ ridge, int parts)
{
    const int m0 = (int)(blockIdx.x / (unsigned)parts) * MR, part = (int)(blockIdx.x % (unsigned)parts);
    double best[MR];
    int bi[MR];
    const double2 *g[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) {
        best[r] = -1.0;
        bi[r] = 0x7fffffff;
        g[r] = G + (size_t)min(m0 + r, nw - 1) * nz;
    }
    for (int n = part * (int)blockDim.x + (int)threadIdx.x; n < nk; n += parts * (int)blockDim.x) {
        double2 acc[MR];
#pragma unroll
        for (int r = 0; r < MR; ++r) acc[r] = make_double2(0.0, 0.0);
#pragma unroll UZ
        for (int z = 0; z < nz; ++z) {
            const double2 e = E[(size_t)z * nk + n];
#pragma unroll
            for (int r = 0; r < MR; ++r) acc[r] = cmul_acc(acc[r], g[r][z], e);
        }
#pragma unroll
        for (int r = 0; r < MR; ++r) {
            if (m0 + r < nw) F[(size_t)(m0 + r) * nk + n] = acc[r];
            const double p = acc[r].x * acc[r].x + acc[r].y * acc[r].y;
            if (p > best[r]) {
                best[r] = p;
                bi[r] = n;
            }
        }
    }
    if (ridge) store_ridge<MR>(best, bi, m0, nw, ridge);
}

// The ridge of one row per workgroup, where the rows are split over workgroups.
__global__ __launch_bounds__(1024) void k_ridge(const double2 *__restrict__ F, int nw, int nk, int *__restrict__ ridge)
{
    double best[1] = {-1.0};
    int bi[1] = {0x7fffffff};
    const double2 *f = F + (size_t)blockIdx.x * nk;
    for (int n = threadIdx.x; n < nk; n += blockDim.x) {
        const double2 v = f[n];
        const double p = v.x * v.x + v.y * v.y;
        if (p > best[0]) {
            best[0] = p;
            bi[0] = n;
        }
    }
    store_ridge<1>(best, bi, (int)blockIdx.x, nw, ridge);
}

// partial sums of x[t][z] exp(-j omega (t0 + t)) over the steps of slice s: one wave per
// (slice, column), lanes over the steps, a fixed-order butterfly across the lanes
__global__ __launch_bounds__(64) void k_harmonic(const double *__restrict__ x, long long nt, int nz, double t0,
                                                 double omega, long long chunk, double2 *__restrict__ ph)
{
    const int z = blockIdx.x, s_ = blockIdx.y;
    const long long ta = (long long)s_ * chunk;
    const long long tb = min(ta + chunk, nt);
    double ar = 0.0, ai = 0.0;
    for (long long t = ta + threadIdx.x; t < tb; t += 64) {
        double s, c;
        sincos(omega * (t0 + (double)t), &s, &c);
        const double v = x[t * nz + z];
        ar = fma(v, c, ar);
        ai = fma(-v, s, ai);
    }
    for (int off = 32; off > 0; off >>= 1) {
        ar += __shfl_xor(ar, off);
        ai += __shfl_xor(ai, off);
    }
    if (threadIdx.x == 0) ph[(size_t)z * gridDim.y + s_] = make_double2(ar, ai);
}

// P[z] = (2 / nt) (sum of the slices in order); log |P| and arg P per column in parallel,
// then one wave unwraps the phases along the columns (64 columns at a time, a scan of their
// steps) and fits the two straight lines (24 columns: 10 us, 17 with one lane for all of it)
constexpr int kFitLds = 2048;

__global__ __launch_bounds__(1024) void k_wave_fit(const double2 *__restrict__ ph, int nslice, long long nt,
                                                  const double *zpos, int nz, double omega, double2 *la,
                                                  double *__restrict__ out)
{
    const double sc = 2.0 / (double)nt;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
    for (int z = wv; z < nz; z += nwv) {
        // one wave per column: lanes over the slices, then a fixed-order butterfly
        double pr = 0.0, pi_ = 0.0;
        for (int q = lane; q < nslice; q += 64) {
            const double2 v = ph[(size_t)z * nslice + q];
            pr += v.x;
            pi_ += v.y;
        }
        for (int off = 32; off > 0; off >>= 1) {
            pr += __shfl_xor(pr, off);
            pi_ += __shfl_xor(pi_, off);
        }
        pr *= sc;
        pi_ *= sc;
        // log |P| is -inf for P = 0: such a column carries no phase and is left out
        if (lane == 0) la[z] = make_double2(log(hypot(pr, pi_)), atan2(pi_, pr));
    }
    // (log |P|, unwrapped phase) per column: in LDS when they fit
    __shared__ double2 s_la[kFitLds];
    __syncthreads();
    if (wv != 0) return;
    double2 *run_la = nz <= kFitLds ? s_la : la;
    const double pi = 3.14159265358979323846;
    const double ninf = -__builtin_inf();
    double sz = 0.0, sm = 0.0, sp = 0.0;
    int cnt = 0;
    {
        double prev = 0.0, run0 = 0.0; // phase and unwrapped phase of the last column used
        for (int zb = 0; zb < nz; zb += 64) {
            const int z = zb + lane;
            const double2 v = z < nz ? la[z] : make_double2(ninf, 0.0);
            const bool use = !(v.x == ninf);
            const unsigned long long bal = __ballot(use), below = bal & ((1ull << lane) - 1ull);
            const int from = below ? 63 - __clzll((long long)below) : 0;
            const double pv = __shfl(v.y, from);
            double d = v.y - (below ? pv : prev);
            if (d > pi) d -= 2.0 * pi;
            else if (d < -pi) d += 2.0 * pi;
            if (cnt == 0 && !below) d = v.y; // the first column used
            if (!use) d = 0.0;
            for (int off = 1; off < 64; off <<= 1) {
                const double u = __shfl_up(d, off);
                if (lane >= off) d += u;
            }
            const double run = run0 + d;
            if (z < nz) run_la[z] = make_double2(v.x, run);
            if (use) {
                sz += zpos[z];
                sm += v.x;
                sp += run;
            }
            if (bal) {
                cnt += __popcll(bal);
                prev = __shfl(v.y, 63 - __clzll((long long)bal));
                run0 = __shfl(run, 63);
            }
        }
    }
    auto sum = [](double v) {
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        return v;
    };
    if (cnt < 2) {
        const double nan = __builtin_nan("");
        if (lane < 6) out[lane] = lane < 5 ? nan : (double)cnt;
        return;
    }
    const double zb = sum(sz) / cnt, mb = sum(sm) / cnt, pb = sum(sp) / cnt;
    double szz = 0.0, szm = 0.0, szp = 0.0;
    for (int z = lane; z < nz; z += 64) { // (each lane the entries that it stored)
        const double2 v = run_la[z];
        if (v.x == ninf) continue;
        const double dz = zpos[z] - zb;
        szz += dz * dz;
        szm += dz * (v.x - mb);
        szp += dz * (v.y - pb);
    }
    szz = sum(szz);
    szm = sum(szm);
    szp = sum(szp);
    if (lane != 0) return;
    const double s_mag = szm / szz, s_ph = szp / szz;
    const double i_mag = mb - s_mag * zb, i_ph = pb - s_ph * zb;
    const double amp = exp(i_mag);
    out[0] = amp * cos(i_ph);
    out[1] = amp * sin(i_ph);
    out[2] = -s_mag;
    out[3] = -s_ph;
    out[4] = omega / (-s_ph);
    out[5] = (double)cnt;
}

// x[i][p] = mean rho' (quantity 0) or sum rho u_z / sum rho (quantity 1) of probe plane p at
// step first + i, from the probe ring records (count, sum rho', sum rho u_z, sum rho)
__global__ __launch_bounds__(256) void k_probe_signal(const double *__restrict__ ring, int ring_len, int nprobe,
                                                      long long first, long long n, int quantity,
                                                      double *__restrict__ x)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * nprobe) return;
    const long long s = i / nprobe;
    const int p = (int)(i % nprobe);
    const long long slot = (first + s) % ring_len;
    const double *rec = ring + (slot * nprobe + p) * 4;
    const double cnt = rec[0];
    x[i] = cnt > 0.0 ? (quantity == 0 ? rec[1] / cnt : rec[2] / rec[3]) : 0.0;
}

// x[i][l] = average of velocity component `component` over the particles of layer l after
// step first + i, from the particle-velocity ring; the members of layer l are
// members[start[l] .. start[l + 1]) in index order (a fixed summation order)
__global__ __launch_bounds__(256) void k_particle_signal(const double *__restrict__ ring, int ring_len, int ptot,
                                                         int p_off, long long first, long long n,
                                                         const int *__restrict__ start,
                                                         const int *__restrict__ members, int n_layers,
                                                         int component, double *__restrict__ x)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * n_layers) return;
    const long long st = i / n_layers;
    const int l = (int)(i - st * n_layers);
    const double *rec = ring + ((first + st) % ring_len) * (long long)ptot * 3;
    const int a = start[l], b = start[l + 1];
    double sum = 0.0;
    for (int k = a; k < b; ++k) sum += rec[(long long)(p_off + members[k]) * 3 + component];
    x[i] = b > a ? sum / (double)(b - a) : 0.0;
}

inline long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }

}  // namespace

DftPlan dft_plan(long long nt, int nz, int nw, int nk)
{
    DftPlan p;
    // the fit's slices: whole waves of steps, about 1024 workgroups' worth of them
    constexpr int kSlice = 64;
    const long long zgroups = ceil_div(nz, 8), zblocks = ceil_div(nz, 8 * std::min<long long>(4, zgroups));
    long long nslice = std::max<long long>(1, 1024 / zblocks);
    nslice = std::min(nslice, std::max<long long>(1, ceil_div(nt, kSlice)));
    p.slice = ceil_div(ceil_div(nt, nslice), kSlice) * kSlice;
    p.nslice = (int)ceil_div(nt, p.slice);
    // the time stage: as many chunks of four segments as fill the chip
    p.nwb = (int)ceil_div(nw, 16 * kMT);
    p.ztiles = nz > 16 ? 2 : 1;
    p.nzb = (int)ceil_div(nz, 16 * p.ztiles);
    long long nchunk = std::max<long long>(1, kTimeBlocks / ((long long)p.nwb * p.nzb));
    nchunk = std::min(nchunk, ceil_div(nt, 4 * 64)); // (at least 64 rows a wave)
    p.seg = ceil_div(ceil_div(nt, 4 * nchunk), 8) * 8;
    p.nchunk = (int)ceil_div(nt, 4 * p.seg);
    const size_t sz2 = sizeof(double2);
    p.part_bytes = (std::max((size_t)p.nchunk * nw, (size_t)p.nslice) * nz * sz2 + 255) / 256 * 256;
    p.g_bytes = ((size_t)nw * nz * sz2 + 255) / 256 * 256;
    p.e_bytes = ((size_t)nz * nk * sz2 + 255) / 256 * 256;
    return p;
}

hipError_t launch_st_dft(const DftPlan &p, const double *x, long long nt, int nz, const double *zpos, double t0,
                         double w0, double dw, int nw, double k0, double dk, int nk, double *F, int *ridge,
                         void *work, hipStream_t st)
{
    char *w = (char *)work;
    double2 *part = (double2 *)w;
    double2 *G = (double2 *)(w + p.part_bytes);
    double2 *E = (double2 *)(w + p.part_bytes + p.g_bytes);
    const dim3 tgrid((unsigned)((long long)p.nwb * p.nchunk), p.nzb);
    if (p.ztiles == 2)
        hipLaunchKernelGGL(k_dft_time<2>, tgrid, dim3(256), 0, st, x, nt, nz, t0, w0, dw, nw, p.nwb, p.seg, part);
    else
        hipLaunchKernelGGL(k_dft_time<1>, tgrid, dim3(256), 0, st, x, nt, nz, t0, w0, dw, nw, p.nwb, p.seg, part);
    const long long nmz = (long long)nw * nz;
    const unsigned sum_blocks = (unsigned)ceil_div(nmz, 256);
    hipLaunchKernelGGL(k_dft_sum, dim3(sum_blocks + (unsigned)ceil_div((long long)nz * nk, 256)), dim3(256), 0, st,
                       (const double2 *)part, nmz, p.nchunk, G, sum_blocks, zpos, nz, k0, dk, nk, E);
    // One workgroup per row leaves CUs without one where rows are few: once a row keeps a CU
    // longer than the launch of a kernel for the ridge takes, it is split over workgroups of 256 n
    // (us per call, one workgroup a row | split: 64 x 1024 x 24 20.5 | 23.7, 16 x 4096 x 24
    // 31.9 | 24.6, 16 x 4096 x 64 57 | 25, 1 x 4096 x 4096 2712 | 285, 1 x 2^20 x 24 7417 | 642;
    // sizes nw x nk x nz).  With few columns a row costs little more than F, which the ridge's
    // kernel would read again: 203 x 71856 x 2 74 | 97.
    // Rows share a load of E as long as a workgroup is left for every CU and enough waves to hide
    // each other's chains of loads (1, 2, 4 rows: 1024 x 64 x 1000 84, 125, 141 us; 600 x 300 x
    // 4096 634, 445, -; 1024 x 256 x 1000 177, 133, 147; 1024 x 1024 x 1000 553, 321, 243).
    const bool split = nw < 2 * kCus && nk > 256 && nz >= 8 && (long long)nz * nk > kSplitRow;
    const dim3 sblock(split ? 256u : (unsigned)std::min<long long>(1024, ceil_div(nk, 64) * 64));
    const long long waves = nw * ceil_div(nk, 64);
    const int mr = (split || nw >= 4 * kCus) && waves >= 64 * kCus ? 4
                 : (split || nw >= 2 * kCus) && waves >= 10 * kCus ? 2 : 1;
    // (with many columns a chain of loads: one row leaves the registers for eight in flight, 16 x
    // 16 x 4096 322 us with four, 200 with eight)
    auto space = mr == 4 ? k_dft_space<4, 4> : (mr == 2 ? k_dft_space<2, 4>
                                                        : (nz >= 32 ? k_dft_space<1, 8> : k_dft_space<1, 4>));
    const int parts = split ? (int)ceil_div(nk, 256) : 1;
    hipLaunchKernelGGL(space, dim3((unsigned)(ceil_div(nw, mr) * parts)), sblock, 0, st, (const double2 *)G,
                       (const double2 *)E, nz, nw, nk, (double2 *)F, split ? nullptr : ridge, parts);
    if (split && ridge)
        hipLaunchKernelGGL(k_ridge, dim3(nw), dim3(1024), 0, st, (const double2 *)F, nw, nk, ridge);
    return hipGetLastError();
}

hipError_t launch_wave_fit(const double *x, long long nt, int nz, const double *zpos, double t0, double omega,
                           double *out, void *work, hipStream_t st)
{
    // the slices' partial sums fill the plan's partials region, the per-column (log |P|, arg P)
    // its time-stage sums region
    const DftPlan p = dft_plan(nt, nz, 1, 1);
    double2 *ph = (double2 *)work;
    double2 *la = (double2 *)((char *)work + p.part_bytes);
    hipLaunchKernelGGL(k_harmonic, dim3(nz, p.nslice), dim3(64), 0, st, x, nt, nz, t0, omega, p.slice, ph);
    hipLaunchKernelGGL(k_wave_fit, dim3(1), dim3(1024), 0, st, (const double2 *)ph, p.nslice, nt, zpos, nz, omega, la,
                       out);
    return hipGetLastError();
}

hipError_t launch_particle_signal(const double *ring, int ring_len, int ptot, int p_off, long long first,
                                  long long n, const int *start, const int *members, int n_layers, int component,
                                  double *x, hipStream_t st)
{
    const long long tot = n * n_layers;
    if (tot == 0) return hipSuccess;
    hipLaunchKernelGGL(k_particle_signal, dim3((unsigned)ceil_div(tot, 256)), dim3(256), 0, st, ring, ring_len, ptot,
                       p_off, first, n, start, members, n_layers, component, x);
    return hipGetLastError();
}

hipError_t launch_probe_signal(const double *ring, int ring_len, int nprobe, long long first, long long n,
                               int quantity, double *x, hipStream_t st)
{
    const long long tot = n * nprobe;
    if (tot == 0) return hipSuccess;
    hipLaunchKernelGGL(k_probe_signal, dim3((unsigned)ceil_div(tot, 256)), dim3(256), 0, st, ring, ring_len, nprobe,
                       first, n, quantity, x);
    return hipGetLastError();
}

// Scratch of the allocation-free fit (lbdem_wave_fit_noalloc): a file-scope device array,
// one copy per GPU held until the process ends.  Host code never uses the array's name as
// an address: its device address is taken once per device with hipGetSymbolAddress (with
// that device current) and kept.  Calls on one GPU share the array, so calls that overlap
// on one GPU race; the fit's kernels write every scratch value before reading it.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

hipError_t noalloc_scratch(void **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

}  // namespace lbdem
