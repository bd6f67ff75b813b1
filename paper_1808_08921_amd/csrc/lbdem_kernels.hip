// lbdem_kernels.hip -- gfx950 kernels of the coupled lattice-Boltzmann / DEM step.
//
// Method: Cheng, Luding, Rivas, Harting, Magnanimo, "Hydro-micromechanical modeling of
// wave propagation in saturated granular media", arXiv 1808.08921, Sec. 2.
//
// Five kernels make one time step t -> t+1 of every lattice of a set, in this order
// (Secs. 2.1-2.4; the paper gives no order: this one lets the particle velocities of the
// step be solved together with the momentum their links exchange in it):
//   k_refresh    brings the node map of step t up to date with the previous re-projection's
//                changes, refreshes the link words of the changed nodes and their
//                neighbours, and rebuilds the node lists (moving the populations of changed
//                planes under compact storage) once a particle may have crossed their skin.
//   k_links      8 or more waves per particle, each for a z-slab of the nodes around it: the
//                link pass.  A slab whose link words changed has its link entries found
//                again first, with their link-set sums (the 6 x 6 matrix Z of the motion
//                kernel comes from them).  With Eq. (mem) substituted, the link force of Eq.
//                (fFS) is 2 c_d f~_d(x,t) minus a term linear in the particle's velocities;
//                per (particle, slab) the first part and its torque (F0, T0) are summed in
//                FP64 from the populations f~(t) at the entries' nodes.
//   k_motion     one wave per particle: contacts (Eqs. fdLawn, fdLaws) at X(t), then the
//                velocities of the step from (M + Z)(V', Omega') = M (V, Omega) + F0 + contacts
//                + F_g + the conversion impulses of the previous re-projection (Eqs. translate,
//                rotate, coupleF, coupleT; implicit in the exchanged momentum), X(t+1).  In a set
//                of few particles a wave of k_links does this.
//   k_fluid      one thread per listed node of a z plane (compact storage, the default), or
//                per node of a dense tile: pull streaming (Eq. stream) with stationary walls,
//                moving half-way bounce-back at the particles' new velocities (Eq. mem), the
//                density faces (Sec. 2.4), BGK collision (Eqs. bgk, BGKequili, rhoAndU) and
//                probe partial sums.
//   k_remap      one wave per particle: re-projects the particle on the lattice (Sec. 2.3)
//                where its motion can have changed a node, converts covered and uncovered
//                nodes (Eqs. convertFS, convertSF) and records the impulses that act in the
//                next step; extra workgroups reduce the probe planes; the step counter
//                advances.
// Populations are SoA, [19][nz][ny][nx] per lattice in the node layout, or per z plane at
// the ranks of the plane's listed nodes under compact storage.  The fluid kernel is bound
// by HBM bandwidth (about 1.5 flop per byte at FP32) and uses no MFMA.
#include "lbdem_internal.hpp"

namespace lbdem {

// D3Q19 velocity set in the paper's order (Eq. 3d19q); index = paper index - 1.
constexpr int kCX[kQ] = {1, -1, 0, 0, 0, 0, 1, 1, 1, 1, -1, -1, -1, -1, 0, 0, 0, 0, 0};
constexpr int kCY[kQ] = {0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1, 0};
constexpr int kCZ[kQ] = {0, 0, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 1, -1, 1, -1, 0};
constexpr int kOPP[kQ] = {1, 0, 3, 2, 5, 4, 11, 10, 13, 12, 7, 6, 9, 8, 17, 16, 15, 14, 18};
// the same components in device memory, for a direction known only at run time
__constant__ int kCXd[kQ] = {1, -1, 0, 0, 0, 0, 1, 1, 1, 1, -1, -1, -1, -1, 0, 0, 0, 0, 0};
__constant__ int kCYd[kQ] = {0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1, 0};
__constant__ int kCZd[kQ] = {0, 0, 0, 0, 1, -1, 0, 0, 1, -1, 0, 0, 1, -1, 1, -1, 1, -1, 0};
// component c_d + 1 of every direction, two bits each: a run-time direction without a load
constexpr unsigned long long pack_dirs(const int (&c)[kQ])
{
    unsigned long long v = 0ull;
    for (int d = 0; d < kQ; ++d) v |= (unsigned long long)(c[d] + 1) << (2 * d);
    return v;
}
__device__ __forceinline__ int dir_x(int d) { return (int)(pack_dirs(kCX) >> (2 * d) & 3ull) - 1; }
__device__ __forceinline__ int dir_y(int d) { return (int)(pack_dirs(kCY) >> (2 * d) & 3ull) - 1; }
__device__ __forceinline__ int dir_z(int d) { return (int)(pack_dirs(kCZ) >> (2 * d) & 3ull) - 1; }
// lattice weights (Sec. 2.1): 1/18 along the axes, 1/36 on the diagonals, 1/3 at rest
constexpr double kWd[kQ] = {1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18,
                            1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                            1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 3};
constexpr double kCS2 = 1.0 / 3.0;
// 2 w_d / c_s^2 of the moving-wall term of Eq. (mem)
constexpr double kMW[kQ] = {2.0 * kWd[0] / kCS2, 2.0 * kWd[1] / kCS2, 2.0 * kWd[2] / kCS2, 2.0 * kWd[3] / kCS2,
                            2.0 * kWd[4] / kCS2, 2.0 * kWd[5] / kCS2, 2.0 * kWd[6] / kCS2, 2.0 * kWd[7] / kCS2,
                            2.0 * kWd[8] / kCS2, 2.0 * kWd[9] / kCS2, 2.0 * kWd[10] / kCS2, 2.0 * kWd[11] / kCS2,
                            2.0 * kWd[12] / kCS2, 2.0 * kWd[13] / kCS2, 2.0 * kWd[14] / kCS2, 2.0 * kWd[15] / kCS2,
                            2.0 * kWd[16] / kCS2, 2.0 * kWd[17] / kCS2, 2.0 * kWd[18] / kCS2};
// 1 / w_d (exact) for the 16-bit deviation codec
constexpr float kInvW[kQ] = {18, 18, 18, 18, 18, 18, 36, 36, 36, 36, 36, 36, 36, 36, 36, 36, 36, 36, 3};

// ---------------------------------------------------------------------------
// storage precisions
// ---------------------------------------------------------------------------
template <int P> struct Prec;
template <> struct Prec<PREC_FP64> { using S = double; using C = double; };
template <> struct Prec<PREC_FP32> { using S = float; using C = float; };
template <> struct Prec<PREC_FP16DEV> { using S = _Float16; using C = float; };
template <> struct Prec<PREC_BF16DEV> { using S = uint16_t; using C = float; };

__device__ __forceinline__ uint16_t f32_to_bf16(float x)
{
    // round to nearest even, one instruction (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(uint16_t, (__bf16)x);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// element idx of an array whose byte size stays below 4 GiB: a 32-bit byte offset from a
// base that is the same in every lane (scalar base + vector offset addressing)
template <typename T>
__device__ __forceinline__ T ldo(const T *base, unsigned idx)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + idx * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void sto(T *base, unsigned idx, T v)
{
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + idx * (unsigned)sizeof(T)) = v;
}

// decode population d from storage: FP64 holds f, FP32 the deviation f - w_d rho_f (the
// rest value rounded once to FP32), the 16-bit forms q = f / w_d - rho_f
template <int P>
__device__ __forceinline__ typename Prec<P>::C ld(const typename Prec<P>::S *a, unsigned idx, int d, double rho_f)
{
    if constexpr (P == PREC_FP64) {
        return ldo(a, idx);
    } else if constexpr (P == PREC_FP32) {
        return ldo(a, idx) + (float)(kWd[d] * rho_f);
    } else if constexpr (P == PREC_FP16DEV) {
        return (float)kWd[d] * ((float)rho_f + (float)ldo(a, idx));
    } else {
        return (float)kWd[d] * ((float)rho_f + bf16_to_f32(ldo(a, idx)));
    }
}
// encode population d to storage
template <int P>
__device__ __forceinline__ void st(typename Prec<P>::S *a, unsigned idx, int d, typename Prec<P>::C f, double rho_f)
{
    using S = typename Prec<P>::S;
    if constexpr (P == PREC_FP64) {
        sto(a, idx, (S)f);
    } else if constexpr (P == PREC_FP32) {
        sto(a, idx, f - (float)(kWd[d] * rho_f));
    } else if constexpr (P == PREC_FP16DEV) {
        sto(a, idx, (S)(f * kInvW[d] - (float)rho_f));
    } else {
        sto(a, idx, f32_to_bf16(f * kInvW[d] - (float)rho_f));
    }
}

// the same for a loaded value, and for a direction known at run time by its weight w
template <int P>
__device__ __forceinline__ typename Prec<P>::C decode_full(typename Prec<P>::S v, int d, double rho_f)
{
    if constexpr (P == PREC_FP64) return v;
    else if constexpr (P == PREC_FP32) return v + (float)(kWd[d] * rho_f);
    else if constexpr (P == PREC_FP16DEV) return (float)kWd[d] * ((float)rho_f + (float)v);
    else return (float)kWd[d] * ((float)rho_f + bf16_to_f32(v));
}
template <int P>
__device__ __forceinline__ void encode_full(typename Prec<P>::S *a, typename Prec<P>::C f, double w, double rho_f)
{
    using S = typename Prec<P>::S;
    const float iw = w > 0.3 ? 3.0f : (w > 0.05 ? 18.0f : 36.0f); // 1 / w_d, exact
    if constexpr (P == PREC_FP64) *a = (S)f;
    else if constexpr (P == PREC_FP32) *a = f - (float)(w * rho_f);
    else if constexpr (P == PREC_FP16DEV) *a = (S)(f * iw - (float)rho_f);
    else *a = f32_to_bf16(f * iw - (float)rho_f);
}

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ int xcd_swizzle(int b, int G)
{
    // blocks are dealt round-robin to the 8 XCDs; give each XCD a contiguous tile range
    const int q = G >> 3, r = G & 7, x = b & 7, k = b >> 3;
    return (x < r) ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

__device__ __forceinline__ int wrapc(int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

__device__ __forceinline__ double mimg(double dx, int per, double n)
{
    if (per) {
        if (dx > 0.5 * n) dx -= n;
        else if (dx < -0.5 * n) dx += n;
    }
    return dx;
}

// Position of fluid node (i, j, k) relative to the image of a particle centre X that holds
// the node's link group grp (directions e whose source x - c_e lies in that image): the
// minimum image of x - X, or, in a set with a narrow periodic lattice (NR), where two
// images can border one node, the minimum image of the first link's midpoint x - c_e / 2
// (always less than half a period from its own image's centre) plus c_e / 2.
template <bool NR>
__device__ __forceinline__ void group_arm(const MemberDev *M, unsigned grp, int i, int j, int k, double X0, double X1,
                                          double X2, double &r0, double &r1, double &r2)
{
    if constexpr (NR) {
        const int e = __ffs(grp) - 1;
        const double h0 = 0.5 * (double)kCXd[e], h1 = 0.5 * (double)kCYd[e], h2 = 0.5 * (double)kCZd[e];
        r0 = mimg(((double)i - h0) - X0, M->per[0], M->box[0]) + h0;
        r1 = mimg(((double)j - h1) - X1, M->per[1], M->box[1]) + h1;
        r2 = mimg(((double)k - h2) - X2, M->per[2], M->box[2]) + h2;
    } else {
        r0 = mimg((double)i - X0, M->per[0], M->box[0]);
        r1 = mimg((double)j - X1, M->per[1], M->box[1]);
        r2 = mimg((double)k - X2, M->per[2], M->box[2]);
    }
}

// Image of particle centre X (per axis -1, 0 or +1 periods, packed 2 bits an axis) that
// holds the source (si, sj, sk) of a link, given unwrapped (it may lie one node outside
// the lattice); 0 on a lattice that is not narrow.
__device__ __forceinline__ int source_image(const MemberDev *M, int si, int sj, int sk, const double *X)
{
    if (!M->narrow) return 0;
    const int s3[3] = {si, sj, sk};
    int code = 0;
    for (int a = 0; a < 3; ++a) {
        int n = 0;
        if (M->per[a]) {
            const double d = (double)s3[a] - X[a];
            n = (d > 0.5 * M->box[a]) ? 1 : (d < -0.5 * M->box[a]) ? -1 : 0;
        }
        code |= (n + 1) << (2 * a);
    }
    return code;
}

__device__ __forceinline__ double dist2(const MemberDev *M, int i, int j, int k, double X0, double X1, double X2)
{
    const double dx = mimg((double)i - X0, M->per[0], M->box[0]);
    const double dy = mimg((double)j - X1, M->per[1], M->box[1]);
    const double dz = mimg((double)k - X2, M->per[2], M->box[2]);
    return (dx * dx + dy * dy) + dz * dz;
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_d(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWMASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWMASK, 0xf, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ int dpp_i(int v, int old)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWMASK, 0xf, false);
}

__device__ __forceinline__ double readlane_d(double v, int l)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes in a fixed order, returned to every lane: DPP sums within each
// row of 16 lanes, then the four row sums are added in row order.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_d<0xB1, 0xF>(v);  // quad_perm [1,0,3,2]
    v += dpp_d<0x4E, 0xF>(v);  // quad_perm [2,3,0,1]
    v += dpp_d<0x141, 0xF>(v); // row_half_mirror
    v += dpp_d<0x140, 0xF>(v); // row_mirror
    return ((readlane_d(v, 0) + readlane_d(v, 16)) + readlane_d(v, 32)) + readlane_d(v, 48);
}
__device__ __forceinline__ int wave_sum_i(int v)
{
    v += dpp_i<0xB1, 0xF>(v, 0);
    v += dpp_i<0x4E, 0xF>(v, 0);
    v += dpp_i<0x141, 0xF>(v, 0);
    v += dpp_i<0x140, 0xF>(v, 0);
    return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
           (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
// Minimum over the 64 lanes of non-negative values (their bit patterns order like the values),
// returned to every lane.
__device__ __forceinline__ double wave_min_d(double v)
{
    long long b = __double_as_longlong(v);
    int hi = (int)(b >> 32);
    unsigned lo = (unsigned)b;
    for (int off = 32; off >= 1; off >>= 1) {
        const int ohi = __shfl_xor(hi, off, 64);
        const unsigned olo = (unsigned)__shfl_xor((int)lo, off, 64);
        if (ohi < hi || (ohi == hi && olo < lo)) { hi = ohi; lo = olo; }
    }
    return __longlong_as_double(((long long)hi << 32) | lo);
}

// Makes a wave's LDS writes visible to its other lanes.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Block-wide (256 threads) sums of N doubles in a fixed order; result valid in thread 0.
template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N], double (*red)[8])
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < N; ++c) v[c] = wave_sum(v[c]);
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < N; ++c) red[wv][c] = v[c];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < N; ++c) v[c] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
    __syncthreads();
}

// values that are the same in every lane, moved to scalar registers
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni(long long v)
{
    const int lo = __builtin_amdgcn_readfirstlane((int)(v & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
    return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double uni(double v) { return __longlong_as_double(uni((long long)__double_as_longlong(v))); }

__device__ __forceinline__ const MemberDev *member_of_tile(const DevSet &s, int g)
{
    int lo = 0, hi = s.nmem - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s.mem[mid].tile_off <= g) lo = mid;
        else hi = mid - 1;
    }
    return s.mem + uni(lo);
}

// Density boundary on a z face: non-equilibrium bounce-back (Sec. 2.4) with zero
// tangential velocity; the velocity normal to the face follows from the density.
template <typename C>
__device__ __forceinline__ void zou_he(C (&f)[kQ], C rho, bool top)
{
    // paper indices k -> f[k-1]
    const C s0 = f[0] + f[1] + f[2] + f[3] + f[6] + f[7] + f[10] + f[11] + f[18];
    const C nxc = C(0.5) * (f[0] + f[6] + f[7] - f[1] - f[10] - f[11]);
    const C nyc = C(0.5) * (f[2] + f[6] + f[10] - f[3] - f[7] - f[11]);
    if (!top) {
        const C sm = f[5] + f[9] + f[13] + f[15] + f[17];
        const C ruz = rho - (s0 + C(2) * sm);
        f[4] = f[5] + ruz / C(3);
        f[8] = f[13] + ruz / C(6) - nxc;
        f[12] = f[9] + ruz / C(6) + nxc;
        f[14] = f[17] + ruz / C(6) - nyc;
        f[16] = f[15] + ruz / C(6) + nyc;
    } else {
        const C sp = f[4] + f[8] + f[12] + f[14] + f[16];
        const C ruz = (s0 + C(2) * sp) - rho;
        f[5] = f[4] - ruz / C(3);
        f[13] = f[8] - ruz / C(6) + nxc;
        f[9] = f[12] - ruz / C(6) - nxc;
        f[17] = f[14] - ruz / C(6) + nyc;
        f[15] = f[16] - ruz / C(6) - nyc;
    }
}

// acc + sign * v, or sign * v when acc holds no term yet (a sum started from 0 would keep
// an addition of 0 that IEEE signed zeros do not let the compiler drop)
template <typename C>
__device__ __forceinline__ void acc_term(C &acc, bool &any, int sign, C v)
{
    if (sign == 0) return;
    if (any) acc = (sign > 0) ? acc + v : acc - v;
    else acc = (sign > 0) ? v : -v;
    any = true;
}

// c_d . u
template <typename C>
__device__ __forceinline__ C cdot(int d, C ux, C uy, C uz)
{
    C cu = C(0);
    bool any = false;
    acc_term(cu, any, kCX[d], ux);
    acc_term(cu, any, kCY[d], uy);
    acc_term(cu, any, kCZ[d], uz);
    return cu;
}

// rho = sum f, j = sum f c (Eq. rhoAndU), summed in direction order
template <typename C>
__device__ __forceinline__ void moments(const C (&f)[kQ], C &rho, C &jx, C &jy, C &jz)
{
    C r = C(0), x = C(0), y = C(0), z = C(0);
    bool ar = false, ax = false, ay = false, az = false;
#pragma unroll
    for (int d = 0; d < kQ; ++d) {
        acc_term(r, ar, 1, f[d]);
        acc_term(x, ax, kCX[d], f[d]);
        acc_term(y, ay, kCY[d], f[d]);
        acc_term(z, az, kCZ[d], f[d]);
    }
    rho = r; jx = x; jy = y; jz = z;
}

// f^eq_d(rho, u), Eq. (BGKequili), in FP64
__device__ __forceinline__ double feq(int d, double rho, double ux, double uy, double uz, double uu)
{
    const double cu = cdot(d, ux, uy, uz), cs2 = kCS2;
    return kWd[d] * rho * (1.0 + cu / cs2 + (cu * cu) / (2.0 * cs2 * cs2) - uu / (2.0 * cs2));
}
// f^eq_d(rho, u) - w_d rho_f with rho = rho_f + drho, Eq. (BGKequili) written for the
// deviation from the rest state: w_d (drho + rho (c.u / c_s^2 + (c.u)^2 / (2 c_s^4) - u.u /
// (2 c_s^2))), with 1 / c_s^2 = 3 as exact factors 3, 9/2 and 3/2 and fused multiply-adds
// (FP64 divisions by c_s^2, about a dozen instructions each and 57 per node, had cost the
// FCC wave case's FP64 step 9 of 207 us and the FP64 adjoint a fifth of its time)
template <typename C>
__device__ __forceinline__ C feq_dev(int d, C drho, C rho, C ux, C uy, C uz, C uu)
{
    const C cu = cdot(d, ux, uy, uz);
    const C uu3 = C(1.5) * uu;
    if constexpr (sizeof(C) == 8) {
        const C poly = __builtin_fma(C(4.5) * cu, cu, __builtin_fma(C(3), cu, -uu3));
        return (C)kWd[d] * __builtin_fma(rho, poly, drho);
    } else {
        const C poly = __builtin_fmaf(C(4.5) * cu, cu, __builtin_fmaf(C(3), cu, -uu3));
        return (C)kWd[d] * __builtin_fmaf(rho, poly, drho);
    }
}

// stored value of population d -> deviation f_d - w_d rho_f (FP32 stores the deviation;
// the 16-bit forms store q = f / w_d - rho_f, so the deviation is w_d q)
template <int P>
__device__ __forceinline__ typename Prec<P>::C decode_dev(typename Prec<P>::S v, int d, double rho_f)
{
    using C = typename Prec<P>::C;
    if constexpr (P == PREC_FP64) return v - (C)(kWd[d] * rho_f);
    else if constexpr (P == PREC_FP32) return v;
    else if constexpr (P == PREC_FP16DEV) return (float)kWd[d] * (float)v;
    else return (float)kWd[d] * bf16_to_f32(v);
}

// deviation f_d - w_d rho_f -> stored value of population d
template <int P>
__device__ __forceinline__ void store_dev(typename Prec<P>::S *a, unsigned idx, int d, typename Prec<P>::C df,
                                          double rho_f)
{
    using S = typename Prec<P>::S;
    using C = typename Prec<P>::C;
    if constexpr (P == PREC_FP64) sto(a, idx, (S)((C)(kWd[d] * rho_f) + df));
    else if constexpr (P == PREC_FP32) sto(a, idx, df);
    else if constexpr (P == PREC_FP16DEV) sto(a, idx, (S)(df * kInvW[d]));
    else sto(a, idx, f32_to_bf16(df * kInvW[d]));
}

// ---------------------------------------------------------------------------
// link words
// ---------------------------------------------------------------------------
__device__ __forceinline__ const MemberDev *member_of_cell(const DevSet &s, long long c)
{
    int lo = 0, hi = s.nmem - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s.mem[mid].cell_off <= c) lo = mid;
        else hi = mid - 1;
    }
    return s.mem + lo;
}

// Storage slot of node (i, j, k) under compact storage: its rank among the listed nodes
// of plane k, from the row table of its 32-node word; -1 when the node is not listed.
__device__ __forceinline__ int slot_of(const DevSet &s, const MemberDev *M, int i, int j, int k)
{
    const uint2 r = s.rt[M->rt_off + ((long long)k * M->ny + j) * M->nw + (i >> 5)];
    const unsigned b = 1u << (i & 31);
    return (r.x & b) ? k * (M->nx * M->ny) + (int)r.y + __popc(r.x & (b - 1u)) : -1;
}

// Storage slot of local node `cell` = (i, j, k): the node itself, or its compact slot.
__device__ __forceinline__ int node_slot(const DevSet &s, const MemberDev *M, int cell, int i, int j, int k)
{
    return s.compact ? slot_of(s, M, i, j, k) : cell;
}

template <typename T>
__device__ __forceinline__ void move_values(const char *src, long long from, char *dst, long long to, long long stride)
{
    const T *a = reinterpret_cast<const T *>(src);
    T *b = reinterpret_cast<T *>(dst);
    // (all loads before the first store: the buffers may alias as far as the compiler knows)
    T v[kQ];
#pragma unroll
    for (int d = 0; d < kQ; ++d) v[d] = a[d * stride + from];
#pragma unroll
    for (int d = 0; d < kQ; ++d) b[d * stride + to] = v[d];
}

// First link word of a solid node (no link directions); the compact copy of a listed node's
// word is the word itself without its overflow bit.
constexpr unsigned long long kSolidWord = 1ull << 63;
__device__ __forceinline__ unsigned long long compact_word(unsigned long long w0)
{
    return w0 == kSolidWord ? w0 : (w0 & ~kSolidWord);
}

// Link words of node (i, j, k) of lattice M from the node map own (this lattice's part):
// for a fluid node x, the directions e whose source x - c_e lies inside a particle and the
// slot (0..3, in the order the particles are met) of the particle owning each source; on
// a narrow lattice a slot is a (particle, image) pair, the image of each source found from
// the particle positions X (the set's array at time t).
__device__ void link_words(const MemberDev *M, const int *own, const double *X, int i, int j, int k,
                           unsigned long long &w0, unsigned long long &w1)
{
    const int nx = M->nx, ny = M->ny, nz = M->nz;
    w0 = 0ull;
    w1 = 0ull;
    if (own[(k * ny + j) * nx + i] >= 0) {
        w0 = kSolidWord;
        return;
    }
    unsigned mask = 0u, lo = 0u, hi = 0u;
    int id[4] = {-1, -1, -1, -1}, img[4] = {0, 0, 0, 0};
    int nid = 0;
    bool over = false;
#pragma unroll 1
    for (int e = 0; e < kQ - 1; ++e) {
        int c[3] = {i - kCXd[e], j - kCYd[e], k - kCZd[e]};
        const int u[3] = {c[0], c[1], c[2]};
        const int dims[3] = {nx, ny, nz};
        bool ok = true;
        for (int a = 0; a < 3; ++a) {
            if (c[a] < 0 || c[a] >= dims[a]) {
                if (M->per[a]) c[a] = c[a] < 0 ? c[a] + dims[a] : c[a] - dims[a];
                else ok = false;
            }
        }
        if (!ok) continue;
        const int o = own[(c[2] * ny + c[1]) * nx + c[0]];
        if (o < 0) continue;
        const int q = o - M->p_off;
        const int im = source_image(M, u[0], u[1], u[2], X + 3 * (long long)o);
        int sl = 0;
        while (sl < nid && (id[sl] != q || img[sl] != im)) ++sl;
        if (sl == nid) {
            if (nid == 4) { over = true; continue; }
            img[nid] = im;
            id[nid++] = q;
        }
        mask |= 1u << e;
        if (sl & 1) lo |= 1u << e;
        if (sl & 2) hi |= 1u << e;
    }
    if (mask == 0u && !over) return;
    w0 = (unsigned long long)mask | ((unsigned long long)lo << 18) |
         ((unsigned long long)max(id[0], 0) << 36) | ((unsigned long long)max(id[1], 0) << 49) |
         ((unsigned long long)(nid > 2) << 62) | ((unsigned long long)over << 63);
    w1 = (unsigned long long)hi | ((unsigned long long)max(id[2], 0) << 18) | ((unsigned long long)max(id[3], 0) << 31);
}

// Directions of slot g and the slot's local particle index, from the two link words.
__device__ __forceinline__ unsigned slot_dirs(unsigned long long w0, unsigned long long w1, int g, int &id)
{
    const unsigned mask = (unsigned)w0 & 0x3ffffu, lo = (unsigned)(w0 >> 18) & 0x3ffffu;
    const unsigned hi = (unsigned)w1 & 0x3ffffu;
    id = (g == 0) ? (int)(w0 >> 36) & 0x1fff : (g == 1) ? (int)(w0 >> 49) & 0x1fff
       : (g == 2) ? (int)(w1 >> 18) & 0x1fff : (int)(w1 >> 31) & 0x1fff;
    return mask & ((g & 1) ? lo : ~lo) & ((g & 2) ? hi : ~hi);
}

// Marks the chunk of q whose z-slab holds plane z.
__device__ __forceinline__ void mark_dirty(const DevSet &s, const MemberDev *M, int q, int z, long long t)
{
    if (q < 0) return;
    const int z0 = s.lzr[2 * q], hz = s.lzr[2 * q + 1];
    if (hz <= 0) return;
    int dz = z - z0;
    if (M->per[2]) dz = ((dz % M->nz) + M->nz) % M->nz;
    if (dz < 0) return;
    const int c = dz / hz;
    if (c < s.chunks) s.ldirty[q * s.chunks + c] = t;
}

// Link words of a node changed (re-projection of the previous step): the cached link
// entries of every particle named in the old or the new words are stale in the chunk that
// holds the node's plane z.
__device__ __forceinline__ void mark_words(const DevSet &s, const MemberDev *M, unsigned long long o0,
                                           unsigned long long o1, unsigned long long n0, unsigned long long n1,
                                           int z, long long stamp)
{
    for (int g = 0; g < 4; ++g) {
        int q;
        if (slot_dirs(o0, o1, g, q) != 0u) mark_dirty(s, M, M->p_off + q, z, stamp);
        if (slot_dirs(n0, n1, g, q) != 0u) mark_dirty(s, M, M->p_off + q, z, stamp);
    }
}

// ---------------------------------------------------------------------------
// fluid kernel
// ---------------------------------------------------------------------------
// FP32 copy of a particle's wall state for the fluid kernel: X, V, Omega, padding
__device__ __forceinline__ void pack_state(float *o, const double *X, const double *V, const double *W)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) { o[a] = (float)X[a]; o[4 + a] = (float)V[a]; o[8 + a] = (float)W[a]; }
    o[3] = o[7] = o[11] = 0.0f;
}

// A lattice's periods as the fluid kernel's moving walls use them, in scalar registers: the
// length of a periodic axis and half of it, infinity on a bounded one (no image is nearer).
// Read from the lattice's constants where they are used, these were six loads waited for one
// after the other in every wave with links.
template <typename C> struct Periods {
    C n[3], half[3];
    int p_off;
};
template <typename C>
__device__ __forceinline__ Periods<C> load_periods(const MemberDev *M)
{
    Periods<C> p;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool per = uni(M->per[a]) != 0;
        p.n[a] = per ? (C)uni(M->box[a]) : C(0);
        p.half[a] = per ? C(0.5) * p.n[a] : (C)__builtin_inf();
    }
    p.p_off = uni(M->p_off);
    return p;
}
template <typename C>
__device__ __forceinline__ C image_of(C dx, C n, C half)
{
    if (dx > half) dx -= n;
    else if (dx < -half) dx += n;
    return dx;
}

// V_b = V + Omega x r for the links of group grp at node (i, j, k) of particle q (a global
// index), in the collision precision C; r is the node's position relative to the image of the
// particle that holds the group (the minimum image, or from a link's midpoint in a set with a
// narrow lattice, as group_arm).  Used with c_d . V_b for the link (x, d), which equals c_d .
// V_b at the link's midpoint since c_d . (Omega x c_d) = 0.  X is the position at time t, V and
// Omega the velocities of the step: the packed FP32 copy (FP32 and 16-bit storage), or the
// FP64 state (written by the motion kernel at the other parity).
template <typename C, bool NR>
__device__ __forceinline__ void slot_velocity(const DevSet &s, const Periods<C> &pd, int q, unsigned grp, int i, int j,
                                              int k, int par, C &u0, C &u1, C &u2)
{
    C x[3], v[3], w[3];
    if constexpr (sizeof(C) == 4) {
        const float4 *pq = reinterpret_cast<const float4 *>(s.pf[par] + 12 * q);
        const float4 a = pq[0], b = pq[1], c = pq[2];
        x[0] = a.x; x[1] = a.y; x[2] = a.z;
        v[0] = b.x; v[1] = b.y; v[2] = b.z;
        w[0] = c.x; w[1] = c.y; w[2] = c.z;
    } else {
        const double *X = s.X[par] + 3 * q, *V = s.V[par ^ 1] + 3 * q, *W = s.W[par ^ 1] + 3 * q;
#pragma unroll
        for (int a = 0; a < 3; ++a) { x[a] = X[a]; v[a] = V[a]; w[a] = W[a]; }
    }
    C h[3] = {C(0), C(0), C(0)};
    if constexpr (NR) {
        const int e = __ffs(grp) - 1;
        h[0] = C(0.5) * (C)dir_x(e); h[1] = C(0.5) * (C)dir_y(e); h[2] = C(0.5) * (C)dir_z(e);
    }
    C r0 = image_of(((C)i - h[0]) - x[0], pd.n[0], pd.half[0]);
    C r1 = image_of(((C)j - h[1]) - x[1], pd.n[1], pd.half[1]);
    C r2 = image_of(((C)k - h[2]) - x[2], pd.n[2], pd.half[2]);
    if constexpr (NR) { r0 += h[0]; r1 += h[1]; r2 += h[2]; }
    u0 = v[0] + (w[1] * r2 - w[2] * r1);
    u1 = v[1] + (w[2] * r0 - w[0] * r2);
    u2 = v[2] + (w[0] * r1 - w[1] * r0);
}

// Eq. (mem) for the links of a fluid node: f_e = f~_d(x,t) - 2 (w_d / c_s^2) rho_f V_b . c_d,
// d = e*, for every direction e whose source is inside a particle; f[e] holds the deviation
// f~_d(x,t) - w_d rho_f (the same relation holds for deviations since w_e = w_d).  V_b comes
// from the particle's position at t and its velocities of the step; the momentum these
// links exchange was accounted for by the link pass and the motion kernel.
template <typename C, bool NR>
__device__ __forceinline__ void moving_wall(const DevSet &s, const Periods<C> &pd, C (&f)[kQ], unsigned long long w0,
                                            int i, int j, int k, int par, double rho_f, long long gc)
{
    const unsigned mask = (unsigned)w0 & 0x3ffffu, lo = (unsigned)(w0 >> 18) & 0x3ffffu;
    const unsigned long long w1 = (w0 >> 62) ? s.lw[s.ncell_total + gc] : 0ull;
    const unsigned hi = (unsigned)w1 & 0x3ffffu;
    // slots 0 and 1 together: both particle states are loaded at once, then every direction
    // takes the velocity of its slot without a branch
    const unsigned g0 = mask & ~lo & ~hi, g1 = mask & lo & ~hi;
    C a0, a1, a2, b0, b1, b2;
    slot_velocity<C, NR>(s, pd, pd.p_off + ((int)(w0 >> 36) & 0x1fff), g0 ? g0 : 1u, i, j, k, par, a0, a1, a2);
    slot_velocity<C, NR>(s, pd, pd.p_off + ((int)(w0 >> 49) & 0x1fff), g1 ? g1 : 1u, i, j, k, par, b0, b1, b2);
    // (the two directions of a pair share 2 (w / c_s^2) rho_f c . V_b up to its sign)
#pragma unroll
    for (int e = 0; e < kQ - 1; ++e) {
        const int d = kOPP[e];
        if (d < e) continue;
        const C m = (C)(kMW[d] * rho_f);
        const C ta = m * cdot(d, a0, a1, a2), tb = m * cdot(d, b0, b1, b2);
        f[e] = f[e] - (((mask & ~hi) >> e) & 1u ? (((lo >> e) & 1u) ? tb : ta) : C(0));
        f[d] = f[d] + (((mask & ~hi) >> d) & 1u ? (((lo >> d) & 1u) ? tb : ta) : C(0));
    }
    // slots 2 and 3 (nodes bordering more than two particles)
    if (hi != 0u) {
#pragma unroll 1
        for (int g = 2; g < 4; ++g) {
            int q;
            const unsigned grp = slot_dirs(w0, w1, g, q);
            if (grp == 0u) continue;
            C u0, u1, u2;
            slot_velocity<C, NR>(s, pd, pd.p_off + q, grp, i, j, k, par, u0, u1, u2);
#pragma unroll
            for (int e = 0; e < kQ - 1; ++e) {
                const int d = kOPP[e];
                const C cu = cdot(d, u0, u1, u2);
                const C m = ((grp >> e) & 1u) ? (C)(kMW[d] * rho_f) : C(0);
                f[e] = f[e] - m * cu;
            }
        }
    }
}

// Start of step t: brings the other node map up to date with the re-projection of step
// t-1 (its change list, or a full copy after an overflow or a particle set-up), refreshes
// the link words of the changed nodes and their neighbours (all of them after a full
// copy) from the node map of step t, and opens the change list of step t.
template <int P>
__global__ __launch_bounds__(256) void k_refresh(DevSet s)
{
    using S = typename Prec<P>::S;
    const long long t = *s.tstep;
    // (both change counts and the list-rebuild step are loaded with the step counter)
    const int cnt0 = s.chgcnt[0], cnt1 = s.chgcnt[1];
    const long long relist_at = *s.relist_at;
    const int par = (int)(t & 1);
    const int cnt = par ? cnt0 : cnt1;
    const bool relist = s.listmode && relist_at == t;
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long t0 = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    bool over = false;
    // (a step that rebuilds the node lists rewrites every compact word in the fluid kernel)
    const bool fix_compact = s.compact && !relist;
    if (cnt > s.chg_cap) {
        // (every link word may change: the fluid kernel rewrites every compact word)
        if (t0 == 0) *s.lwc_bad = t;
        for (long long c = t0; c < s.ncell_total; c += stride) {
            s.own[par ^ 1][c] = s.own[par][c];
            const MemberDev *M = member_of_cell(s, c);
            const int cell = (int)(c - M->cell_off);
            const int nxy = M->nx * M->ny;
            const int k = cell / nxy, rem = cell - k * nxy, j = rem / M->nx, i = rem - j * M->nx;
            unsigned long long w0, w1;
            link_words(M, s.own[par] + M->cell_off, s.X[par], i, j, k, w0, w1);
            const unsigned long long o0 = s.lw[c], o1 = s.lw[s.ncell_total + c];
            if (o0 != w0 || o1 != w1) mark_words(s, M, o0, o1, w0, w1, k, t - 1);
            s.lw[c] = w0;
            s.lw[s.ncell_total + c] = w1;
            over |= (w0 & kSolidWord) != 0ull && w0 != kSolidWord;
        }
    } else {
        const int *lst = s.chg[par ^ 1];
        for (long long e = t0; e < cnt; e += stride) s.own[par ^ 1][lst[2 * e]] = lst[2 * e + 1];
        // the words of the changed nodes and their neighbours: one group of 32 lanes per
        // word, lane e < 18 reading the owner of source e and lane 18 the node's own (one
        // round of loads), every lane assembling the word from the group's values as
        // link_words does, lane 0 storing it
        const int lane = threadIdx.x & 31;
        const long long grp = t0 >> 5, ngrp = stride >> 5;
        for (long long w = grp; w < (long long)cnt * kQ; w += ngrp) {
            const long long ch = w / kQ;
            const int q = (int)(w - ch * kQ); // 18: the changed node itself
            const long long gcell = lst[2 * ch];
            const MemberDev *M = member_of_cell(s, gcell);
            const int nx = M->nx, ny = M->ny, nz = M->nz;
            const int c0 = (int)(gcell - M->cell_off);
            const int k0 = c0 / (nx * ny), rem = c0 - k0 * nx * ny, j0 = rem / nx, i0 = rem - j0 * nx;
            // a neighbour across a bounded face wraps to a node whose words are unchanged;
            // recomputing them is harmless
            const int ci = wrapc(i0 + kCXd[q], nx), cj = wrapc(j0 + kCYd[q], ny), ck = wrapc(k0 + kCZd[q], nz);
            const int *own = s.own[par] + M->cell_off;
            // the node's current words, loaded with the owners (lane 0 compares and stores)
            const long long gc = M->cell_off + (ck * ny + cj) * nx + ci;
            unsigned long long o0 = 0ull, o1 = 0ull;
            if (lane == 0) { o0 = s.lw[gc]; o1 = s.lw[s.ncell_total + gc]; }
            int o = -1, im = 0;
            if (lane < kQ - 1) {
                const int si = ci - kCXd[lane], sj = cj - kCYd[lane], sk = ck - kCZd[lane];
                const bool ok = (M->per[0] || (si >= 0 && si < nx)) && (M->per[1] || (sj >= 0 && sj < ny)) &&
                                (M->per[2] || (sk >= 0 && sk < nz));
                if (ok) o = own[(wrapc(sk, nz) * ny + wrapc(sj, ny)) * nx + wrapc(si, nx)];
                if (o >= 0) im = source_image(M, si, sj, sk, s.X[par] + 3 * (long long)o);
            } else if (lane == kQ - 1) {
                o = own[(ck * ny + cj) * nx + ci];
            }
            const int self = __shfl(o, kQ - 1, 32);
            unsigned mask = 0u, slo = 0u, shi = 0u;
            int id0 = -1, id1 = -1, id2 = -1, id3 = -1;
            bool ov = false;
            if (self < 0) {
                // (on a narrow lattice a slot is a (particle, image) pair: the key packs both)
                for (int e = 0; e < kQ - 1; ++e) {
                    const int oe = __shfl(o, e, 32);
                    if (oe < 0) continue;
                    const int pq = (oe - M->p_off) | (__shfl(im, e, 32) << 24);
                    int sl;
                    if (id0 < 0 || id0 == pq) { id0 = pq; sl = 0; }
                    else if (id1 < 0 || id1 == pq) { id1 = pq; sl = 1; }
                    else if (id2 < 0 || id2 == pq) { id2 = pq; sl = 2; }
                    else if (id3 < 0 || id3 == pq) { id3 = pq; sl = 3; }
                    else { ov = true; continue; }
                    mask |= 1u << e;
                    if (sl & 1) slo |= 1u << e;
                    if (sl & 2) shi |= 1u << e;
                }
            }
            unsigned long long w0 = self >= 0 ? kSolidWord : 0ull, w1 = 0ull;
            if (mask != 0u || ov) {
                w0 = (unsigned long long)mask | ((unsigned long long)slo << 18) |
                     ((unsigned long long)(max(id0, 0) & 0x1fff) << 36) |
                     ((unsigned long long)(max(id1, 0) & 0x1fff) << 49) |
                     ((unsigned long long)(id2 >= 0) << 62) | ((unsigned long long)ov << 63);
                w1 = (unsigned long long)shi | ((unsigned long long)(max(id2, 0) & 0x1fff) << 18) |
                     ((unsigned long long)(max(id3, 0) & 0x1fff) << 31);
            }
            // a changed word marks the chunk at plane ck of every particle it names,
            // old or new: lane l < 8 takes slot l & 3 of the old (l < 4) or the new words, so
            // the particles' chunk layouts are loaded in one round
            const unsigned long long g0w = __shfl(o0, 0, 32), g1w = __shfl(o1, 0, 32);
            if ((g0w != w0 || g1w != w1) && lane < 8) {
                int q;
                const unsigned dirs = (lane < 4) ? slot_dirs(g0w, g1w, lane & 3, q) : slot_dirs(w0, w1, lane & 3, q);
                if (dirs != 0u) mark_dirty(s, M, M->p_off + q, ck, t - 1);
            }
            // the node's compact word at its storage slot, when listed
            const int ns = fix_compact ? node_slot(s, M, (ck * ny + cj) * nx + ci, ci, cj, ck) : -1;
            if (lane == 0) {
                s.lw[gc] = w0;
                s.lw[s.ncell_total + gc] = w1;
                if (ns >= 0) s.lwc[M->cell_off + ns] = compact_word(w0);
                over |= ov;
            }
        }
    }
    if (over) atomicOr(s.flags, 0x80u);

    // node lists, when a particle has moved the skin since they were built (or after a
    // set-up): per z plane, in x-fastest order, every fluid node and every solid node
    // less than the skin inside its particle's surface.  Only such a node can become
    // fluid before a particle has moved the skin.  The skin follows the lattice's
    // fastest particle (kSkinSteps of its last step, within [kSkinMin, kListSkin]).
    if (relist) {
        // One workgroup per plane.  A rebuild is a chain of memory latencies, so each thread
        // scans kScanCells cells at a time with their loads together and one barrier, a node's
        // 19 values are loaded before the first is stored, nodes ahead of the first change of
        // the list stay where they are, and the row tables' running counts come from one scan
        // over the workgroup (settling suspension, FP32, 340 -> 115 us per rebuild; two or four
        // nodes' values in flight per thread 237 and 191 us, for their registers).
        constexpr int kScanCells = 4;
        using U = typename std::conditional<sizeof(S) == 8, unsigned long long,
                                            typename std::conditional<sizeof(S) == 4, unsigned, unsigned short>::type>::type;
        __shared__ int cnt16[2][4 * kScanCells];
        __shared__ double vred[4];
        __shared__ unsigned tab[kMaxPlaneWords];
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
        for (long long q = t0; q < s.ptot; q += stride)
            for (int ax = 0; ax < 3; ++ax) s.Xl[3 * q + ax] = s.X[par][3 * q + ax];
        for (int pl = blockIdx.x; pl < s.nplanes; pl += gridDim.x) {
            int lo = 0, hi = s.nmem - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s.mem[mid].pz_off <= pl) lo = mid;
                else hi = mid - 1;
            }
            const MemberDev *M = s.mem + lo;
            const int z = pl - M->pz_off, nx = M->nx, nxy = M->nx * M->ny;
            const int *own = s.own[par] + M->cell_off;
            int *lst = s.clist + M->cell_off + (long long)z * nxy;
            // the lattice's largest particle step (non-negative: bit patterns order)
            double vm = 0.0;
            for (int q = threadIdx.x; q < M->np; q += blockDim.x) vm = fmax(vm, s.pspd[M->p_off + q]);
            for (int off = 32; off >= 1; off >>= 1) vm = fmax(vm, __shfl_xor(vm, off, 64));
            __syncthreads();
            if (lane == 0) vred[wv] = vm;
            const int ny = M->ny, nw = M->nw;
            if (s.compact)
                for (int w = threadIdx.x; w < ny * nw; w += 256) tab[w] = 0u;
            __syncthreads();
            vm = fmax(fmax(vred[0], vred[1]), fmax(vred[2], vred[3]));
            const double skin = fmin(fmax(kSkinSteps * vm, kSkinMin), kListSkin);
            if (threadIdx.x == 0) s.skin[lo] = skin;
            const int oldcnt = s.ccnt[pl];
            int count = 0;
            int first = 0x7fffffff; // first entry of the list that differs from the previous one
            for (int c0 = 0, buf = 0; c0 < nxy; c0 += 256 * kScanCells, buf ^= 1) {
                int o[kScanCells];
                double R[kScanCells], X[kScanCells][3];
                unsigned long long bal[kScanCells];
#pragma unroll
                for (int u = 0; u < kScanCells; ++u)
                    o[u] = own[z * nxy + min(c0 + 256 * u + (int)threadIdx.x, nxy - 1)];
                if (s.ptot > 0) {
#pragma unroll
                    for (int u = 0; u < kScanCells; ++u) {
                        const int q = max(o[u], 0);
                        R[u] = s.R[q];
                        for (int ax = 0; ax < 3; ++ax) X[u][ax] = s.X[par][3 * q + ax];
                    }
                }
#pragma unroll
                for (int u = 0; u < kScanCells; ++u) {
                    const int c = c0 + 256 * u + (int)threadIdx.x;
                    const int j = c / nx, i = c - j * nx;
                    bool listed = c < nxy;
                    if (listed && o[u] >= 0) {
                        const double rr = R[u] - skin;
                        listed = rr <= 0.0 || dist2(M, i, j, z, X[u][0], X[u][1], X[u][2]) > rr * rr;
                    }
                    if (listed && s.compact) atomicOr(&tab[j * nw + (i >> 5)], 1u << (i & 31));
                    bal[u] = __ballot(listed);
                    if (lane == 0) cnt16[buf][4 * u + wv] = __popcll(bal[u]);
                }
                // (two buffers: a wave may be a round ahead of the others' reads)
                __syncthreads();
                int at[kScanCells], old[kScanCells];
                int run = count;
#pragma unroll
                for (int u = 0; u < kScanCells; ++u)
                    for (int w = 0; w < 4; ++w) {
                        if (w == wv) at[u] = run + __popcll(bal[u] & ((1ull << lane) - 1ull));
                        run += cnt16[buf][4 * u + w];
                    }
                count = run;
#pragma unroll
                for (int u = 0; u < kScanCells; ++u) old[u] = ((bal[u] >> lane) & 1ull) ? lst[at[u]] : 0;
#pragma unroll
                for (int u = 0; u < kScanCells; ++u) {
                    if (!((bal[u] >> lane) & 1ull)) continue;
                    const int cell = z * nxy + c0 + 256 * u + (int)threadIdx.x;
                    if (at[u] >= oldcnt || old[u] != cell) first = min(first, at[u]);
                    lst[at[u]] = cell;
                }
            }
            for (int off = 32; off >= 1; off >>= 1) first = min(first, __shfl_xor(first, off, 64));
            __syncthreads();
            if (lane == 0) cnt16[0][wv] = first;
            __threadfence_block();
            __syncthreads();
            first = min(min(cnt16[0][0], cnt16[0][1]), min(cnt16[0][2], cnt16[0][3]));
            first = min(first, count);
            // compact storage: an unchanged list keeps its slots, nothing moves
            const bool moved = first < count || count != oldcnt;
            if (threadIdx.x == 0) s.ccnt[pl] = count;
            if (s.compact && moved) {
                // compact storage: move the plane's populations to the new list order
                // (through the scratch buffer), then rewrite the plane's row tables
                const long long nc = M->ncell, po = M->pop_off * (long long)s.es;
                char *A = (char *)(par ? s.popB : s.popA) + po;
                char *Cb = (char *)s.popC + po;
                for (int k = first + (int)threadIdx.x; k < count; k += 256) {
                    const int c = lst[k] - z * nxy, j = c / nx, i = c - j * nx;
                    const int old = slot_of(s, M, i, j, z);
                    const long long to = (long long)z * nxy + k;
                    if (old < 0) {
                        // not listed before: a node uncovered in the last re-projection
                        // takes its parked refill f^eq(rho_bar, V_b) (Eq. convertSF); any
                        // other is solid and takes the rest state w_d rho_f until refilled
                        const long long gcell = M->cell_off + lst[k];
                        const int pi = s.pend[gcell];
                        double rb = M->rho_f, u0 = 0.0, u1 = 0.0, u2 = 0.0;
                        if (pi >= 0) {
                            const double *rec = s.pbuf[par ^ 1] + 4 * pi;
                            rb = rec[0]; u0 = rec[1]; u1 = rec[2]; u2 = rec[3];
                            s.pend[gcell] = -1;
                        }
                        const double uu = u0 * u0 + u1 * u1 + u2 * u2;
                        S *CbS = reinterpret_cast<S *>(Cb);
                        for (int d = 0; d < kQ; ++d)
                            st<P>(CbS, (unsigned)(d * nc + to), d, (typename Prec<P>::C)feq(d, rb, u0, u1, u2, uu),
                                  M->rho_f);
                        continue;
                    }
                    move_values<U>(A, old, Cb, to, nc);
                }
                // (every thread has read the old tables)
                __threadfence_block();
                __syncthreads();
                {
                    const int nwords = ny * nw, per = (nwords + 255) / 256;
                    const int w0 = min((int)threadIdx.x * per, nwords), w1 = min(w0 + per, nwords);
                    int sum = 0;
                    for (int w = w0; w < w1; ++w) sum += __popc(tab[w]);
                    int run = sum;
                    for (int off = 1; off < 64; off <<= 1) {
                        const int up = __shfl_up(run, off, 64);
                        if (lane >= off) run += up;
                    }
                    if (lane == 63) cnt16[1][wv] = run;
                    __syncthreads();
                    run -= sum;
                    for (int w = 0; w < wv; ++w) run += cnt16[1][w];
                    uint2 *rtp = s.rt + M->rt_off + (long long)z * nwords;
                    for (int w = w0; w < w1; ++w) {
                        rtp[w] = make_uint2(tab[w], (unsigned)run);
                        run += __popc(tab[w]);
                    }
                }
                for (int k = first + (int)threadIdx.x; k < count; k += 256) {
                    const long long at = (long long)z * nxy + k;
                    move_values<U>(Cb, at, A, at, nc);
                }
                __threadfence_block();
                __syncthreads();
            }
        }
    }
    if (t0 == 0) {
        s.chgcnt[par] = 0;
        s.pcnt[par] = 0; // parked refills of this step's re-projection
        *s.tcopy = t; // the re-projection kernel of this step reads the step from here
    }
}

// Pull streaming (Eq. stream), stationary half-way walls, moving half-way walls on the
// particles (Eq. mem, from the node's link words), the density faces (Sec. 2.4), BGK
// collision (Eqs. bgk, BGKequili, rhoAndU) and probe partial sums.
template <int P, bool CMP, bool NR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(P == PREC_FP64 ? 3 : (CMP ? 6 : 5)))) void k_fluid(DevSet s)
{
    using S = typename Prec<P>::S;
    using C = typename Prec<P>::C;
    __shared__ double red[4][8];

    const long long t = *s.tstep;
    const int par = (int)(t & 1);
    const int g = xcd_swizzle(blockIdx.x, gridDim.x);
    const MemberDev *M = member_of_tile(s, g);
    const int tl = g - uni(M->tile_off);
    const int ntx = uni(M->ntx), nty = uni(M->nty);
    const int nx = uni(M->nx), ny = uni(M->ny), nz = uni(M->nz);
    const int nc = (int)uni(M->ncell);
    const int nxy = nx * ny;
    const long long pop_off = uni(M->pop_off), cell_off = uni(M->cell_off);
    const int pz_off = uni(M->pz_off);
    const S *A = (const S *)(par ? s.popB : s.popA) + pop_off;
    S *B = (S *)(par ? s.popA : s.popB) + pop_off;
    const double rho_fd = uni(M->rho_f);
    const C omega = (C)uni(M->omega);
    const int bc4 = uni(M->bc[4]), bc5 = uni(M->bc[5]);
    // (the rest of the lattice's constants are read here too: the barriers of the node
    // loop below would otherwise make each wave read them again after them)
    const int bc0 = uni(M->bc[0]), bc1 = uni(M->bc[1]), bc2 = uni(M->bc[2]), bc3 = uni(M->bc[3]);
    const long long rt_off = CMP ? uni(M->rt_off) : 0ll;
    const int nw = CMP ? uni(M->nw) : 0, per_x = uni(M->per[0]);
    const long long t_n = uni(M->t_n);
    long long ti = t + 1;
    if (ti > t_n + 1) ti = t_n + 1;
    const C drho_in = (C)(s.wave[uni(M->wave_off) + ti] - rho_fd);
    const Periods<C> pd = load_periods<C>(M);
    // compact storage: every listed node's compact word is written here after a list rebuild
    // or a full copy of the node map, and read from its slot otherwise
    const bool full_compact = CMP && (*s.relist_at == t || *s.lwc_bad == t);

    // CMP: compact storage (node lists, populations at the nodes' ranks in the lists)
    const bool lists = CMP || s.listmode != 0;
    constexpr bool compact = CMP;

    // the collision of a fluid node's pulled deviations f, stored at slot me; the node's probe
    // terms and the watchdog: a fluid node whose density is not a positive finite number
    // (status 0x400; NaN fails the first comparison)
    auto collide = [&](const C (&f)[kQ], bool fl, double (&pr)[4], auto &&put) {
        C drho, jx, jy, jz;
        moments<C>(f, drho, jx, jy, jz);
        const C rho = (C)rho_fd + drho;
        if (fl && !(rho > C(0) && rho < C(1e30))) atomicOr(s.flags, 0x400u);
        if (fl) {
            pr[0] = 1.0;
            pr[1] = (double)drho;
            pr[2] = (double)jz;
            pr[3] = rho_fd + (double)drho;
        }
        C ux, uy, uz, uu;
        if constexpr (sizeof(C) == 8) {
            ux = jx / rho; uy = jy / rho; uz = jz / rho;
            uu = ux * ux + uy * uy + uz * uz;
        } else {
            const C ir = C(1) / rho;
            ux = jx * ir; uy = jy * ir; uz = jz * ir;
            uu = __builtin_fmaf(ux, ux, __builtin_fmaf(uy, uy, uz * uz));
        }
#pragma unroll
        for (int d = 0; d < kQ; ++d) {
            const C fe = feq_dev<C>(d, drho, rho, ux, uy, uz, uu);
            C post;
            if constexpr (sizeof(C) == 8) post = f[d] + omega * (fe - f[d]);
            else post = __builtin_fmaf(omega, fe - f[d], f[d]);
            put(d, post);
        }
    };
    // the workgroup's probe sums of plane z0 + dz of its tile; accum adds them to those of an
    // earlier chunk of the same workgroup
    auto probes = [&](int z, int dz, bool accum, double (&v)[4]) {
        if (s.pzmap[pz_off + z] < 0) return;
        block_sum<4>(v, red);
        if (threadIdx.x == 0) {
            double *o = s.pprt + ((long long)g * s.nzt + dz) * 4;
            if (accum) { o[0] += v[0]; o[1] += v[1]; o[2] += v[2]; o[3] += v[3]; }
            else { o[0] = v[0]; o[1] = v[1]; o[2] = v[2]; o[3] = v[3]; }
        }
    };

    // one node (i, j, z) of a dense tile or a node list, at slot me0 under compact storage; word
    // is its first link word
    // compact storage: the row-table words of the workgroup's source rows, staged in LDS
    // (rows j0 - 1 .. j1 + 1 of planes z - 1, z, z + 1 for the chunk's nodes in rows j0 .. j1)
    __shared__ uint2 rt_lds[kRtLds];
    __shared__ int jr[2];

    auto node = [&](int i, int j, int z, int me0, bool vij, const uint2 *lrt, int jb, int nrows,
                    unsigned long long word, double (&pr)[4]) {
        // offsets to the x-1 / x+1 / y-1 / y+1 neighbours (wrapped on periodic axes) and the
        // kind of face crossed to reach them (0 inside or periodic, 1 wall, 2 density face)
        int oxm = (i > 0) ? -1 : (nx - 1), oxp = (i < nx - 1) ? 1 : -(nx - 1);
        int kxm = (i > 0) ? 0 : bc0, kxp = (i < nx - 1) ? 0 : bc1;
        int oym = (j > 0) ? -nx : (ny - 1) * nx, oyp = (j < ny - 1) ? nx : -(ny - 1) * nx;
        int kym = (j > 0) ? 0 : bc2, kyp = (j < ny - 1) ? 0 : bc3;

        {
            // keep the 18 per-direction offsets from being hoisted out of the loop: they are
            // cheap to recompute and would otherwise stay live in 36 registers
            asm volatile("" : "+v"(oxm), "+v"(oxp), "+v"(oym), "+v"(oyp), "+v"(kxm), "+v"(kxp), "+v"(kym), "+v"(kyp));
            const int cell = (z * ny + j) * nx + i;
            const bool fl = vij && word != kSolidWord;
            // Dense tiles with 4- and 8-byte storage write every node of a row, so each store
            // covers whole cache lines: a solid node loads nothing and stores the rest state
            // w_d, a value that is never read (a node is refilled on uncovering).  16-bit
            // storage measured faster with solid nodes left out; with node lists only the
            // fluid nodes work.
            constexpr bool kWholeRows = sizeof(S) >= 4;
            if ((kWholeRows && !lists) ? vij : fl) {
                const int ozm = (z > 0) ? -nxy : (nz - 1) * nxy, ozp = (z < nz - 1) ? nxy : -(nz - 1) * nxy;
                const int kzm = (z > 0) ? 0 : bc4, kzp = (z < nz - 1) ? 0 : bc5;
                // Loads are issued for every lane, a solid lane reading the first element of the
                // array (one shared line) instead of branching around each load.
                const unsigned long long lwv = fl ? word : 0ull;
                const unsigned lmask = (unsigned)lwv & 0x3ffffu;
                // storage slot of this node: the node itself, or its rank in the plane's list
                // (as an offset from the node that the compiler cannot see through: it keeps
                // the register allocation of the node-layout kernel, which has no spills)
                int dlt = compact ? me0 - cell : 0;
                if (compact) asm volatile("" : "+v"(dlt));
                const int me = cell + dlt;
                // compact storage: slots of the sources from the row tables of the 9 source rows
                // (y - c_y, z - c_z).  Along a row the listed nodes hold consecutive slots, so
                // the source x - 1 sits one slot below the node's rank in that row and x + 1
                // one above it (plus one when x itself is listed); a source across a periodic
                // x face reads the table word at the other end of the row.
                int src[kQ - 1];
                if (compact) {
                    const uint2 *rtab = s.rt + rt_off;
                    const unsigned b = 1u << (i & 31);
                    const int wx = (i == 0) ? nx - 1 : 0;
                    const unsigned bw = 1u << (wx & 31);
                    uint2 wv[9], ww[9];
                    if (lrt) {
    #pragma unroll
                        for (int r = 0; r < 9; ++r) {
                            const int row = ((r % 3) * nrows + (j + r / 3 - 1 - jb)) * nw;
                            wv[r] = lrt[row + (i >> 5)];
                            ww[r] = per_x ? lrt[row + (wx >> 5)] : make_uint2(0u, 0u);
                        }
                    } else {
    #pragma unroll
                        for (int r = 0; r < 9; ++r) {
                            const int jj = wrapc(j + r / 3 - 1, ny), zz = wrapc(z + r % 3 - 1, nz);
                            const long long row = ((long long)zz * ny + jj) * nw;
                            wv[r] = rtab[row + (i >> 5)];
                            ww[r] = per_x ? rtab[row + (wx >> 5)] : make_uint2(0u, 0u);
                        }
                    }
    #pragma unroll
                    for (int e = 0; e < kQ - 1; ++e) {
                        const int r = (1 - kCY[e]) * 3 + (1 - kCZ[e]);
                        // (the staged words hold slots, the tables ranks within the plane)
                        const int zb = lrt ? 0 : wrapc(z - kCZ[e], nz) * nxy;
                        const int rk = zb + (int)wv[r].y + __popc(wv[r].x & (b - 1u));
                        const int rwr = zb + (int)ww[r].y + __popc(ww[r].x & (bw - 1u));
                        int v;
                        if (kCX[e] == 0) v = rk;
                        else if (kCX[e] < 0) v = (i < nx - 1) ? rk + ((wv[r].x & b) ? 1 : 0) : rwr;
                        else v = (i > 0) ? rk - 1 : rwr;
                        src[e] = max(v, 0);
                    }
                }
                C f[kQ];
                S raw[kQ];
                unsigned unk = 0u;
    #pragma unroll
                for (int e = 0; e < kQ - 1; ++e) {
                    int off = 0, kind = 0;
                    if (kCX[e] > 0) { off += oxm; kind = max(kind, kxm); } else if (kCX[e] < 0) { off += oxp; kind = max(kind, kxp); }
                    if (kCY[e] > 0) { off += oym; kind = max(kind, kym); } else if (kCY[e] < 0) { off += oyp; kind = max(kind, kyp); }
                    if (kCZ[e] > 0) { off += ozm; kind = max(kind, kzm); } else if (kCZ[e] < 0) { off += ozp; kind = max(kind, kzp); }
                    // f_e(x, t+1) = f~_e(x - c_e, t); from a wall or a particle the population
                    // comes back from this node, f~_{e*}(x, t); across a density face it is unknown
                    const bool back = (kind != 0) || ((lmask >> e) & 1u);
                    // (offsets from array e: the select is taken between per-lane offsets, so
                    // that no per-lane multiply by nc is formed)
                    const unsigned from = compact ? (unsigned)src[e] : (unsigned)(cell + off);
                    const unsigned idx = (unsigned)(e * nc) +
                                         (back ? (unsigned)((kOPP[e] - e) * nc) + (unsigned)me : from);
                    raw[e] = ldo(A, fl ? idx : 0u);
                    unk |= (kind == BC_PRESSURE) ? (1u << e) : 0u;
                }
                raw[18] = ldo(A, fl ? (unsigned)(18 * nc) + (unsigned)me : 0u);
                // the arithmetic works on deviations f_d - w_d rho_f from the rest state: Eqs.
                // (stream), (mem) and the density faces are affine with the same coefficients
                // for f and its deviation (w_d = w_{d*}; the weights of each Zou-He closure sum
                // to one), and the deviations keep the small density and momentum signals
                // clear of the rounding of the O(1) rest populations
    #pragma unroll
                for (int e = 0; e < kQ; ++e)
                    f[e] = (fl && !((unk >> e) & 1u)) ? decode_dev<P>(raw[e], e, rho_fd) : C(0);
                if (lmask != 0u) moving_wall<C, NR>(s, pd, f, lwv, i, j, z, par, rho_fd, cell_off + cell);

                if (z == 0 && bc4 == BC_PRESSURE) zou_he<C>(f, drho_in, false);
                if (z == nz - 1 && bc5 == BC_PRESSURE) zou_he<C>(f, C(0), true);

                collide(f, fl, pr, [&](int d, C post) {
                    store_dev<P>(B, (unsigned)(d * nc) + (unsigned)me, d, post, rho_fd);
                });
            }
        }
    };

    // compact storage, a node away from walls and density faces (periodic faces included) with
    // its source rows staged: along a source row the slots of x - 1, x and x + 1 are the number
    // of listed nodes before x, less one, itself, and with x counted, so a row costs two
    // bit counts, and a wave that holds nodes at a periodic x face reads the row's other end.
    // Fewer vector instructions than the general path, which bound 16-bit storage (FCC wave
    // case, FP16, 35.0 -> 33.0 us per launch); FP32 and FP64 are bound by their traffic (38
    // and 79 us either way, 85 % of the rate of a device copy; an ensemble of 16 lattices in
    // FP32 256 us without and 260 us with it), so they take the general path.
    auto compact_node = [&](int i, int j, int z, int me, bool v, const uint2 *lrt, int jb, int nrows,
                            unsigned long long word, double (&pr)[4]) {
        const bool fl = v && word != kSolidWord;
        // (a lane without a fluid node reads its own slot in every direction)
        const unsigned lmask = fl ? (unsigned)word & 0x3ffffu : 0u, back = fl ? lmask : 0x3ffffu;
        const unsigned below = (1u << (i & 31)) - 1u, upto = 2u * below + 1u;
        const uint2 *row = lrt + (j - 1 - jb) * nw;
        int rk[9], rm[9], rp[9]; // slots of the sources at x, x - 1 and x + 1
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            const uint2 w = row[((r % 3) * nrows + r / 3) * nw + (i >> 5)];
            rk[r] = (int)w.y + __popc(w.x & below);
            if (r % 3 != 1 && r / 3 != 1) continue; // (no direction has c_x, c_y and c_z)
            rm[r] = rk[r] - 1;
            rp[r] = (int)w.y + __popc(w.x & upto);
        }
        if (per_x && __ballot(i == 0 || i == nx - 1) != 0ull) {
            const int wx = (i == 0) ? nx - 1 : 0;
            const unsigned bw = (1u << (wx & 31)) - 1u;
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                if (r % 3 != 1 && r / 3 != 1) continue;
                const uint2 w = row[((r % 3) * nrows + r / 3) * nw + (wx >> 5)];
                const int rw = (int)w.y + __popc(w.x & bw);
                rm[r] = (i == 0) ? rw : rm[r];
                rp[r] = (i == nx - 1) ? rw : rp[r];
            }
        }
        C f[kQ];
        S raw[kQ];
#pragma unroll
        for (int e = 0; e < kQ - 1; ++e) {
            const int r = (1 - kCY[e]) * 3 + (1 - kCZ[e]);
            const int from = kCX[e] == 0 ? rk[r] : (kCX[e] > 0 ? rm[r] : rp[r]);
            raw[e] = ldo(A, ((back >> e) & 1u) ? (unsigned)(kOPP[e] * nc + me) : (unsigned)(e * nc + from));
        }
        raw[18] = ldo(A, (unsigned)(18 * nc + me));
#pragma unroll
        for (int e = 0; e < kQ; ++e) f[e] = decode_dev<P>(raw[e], e, rho_fd);
        if (lmask != 0u)
            moving_wall<C, NR>(s, pd, f, word, i, j, z, par, rho_fd, cell_off + (z * ny + j) * nx + i);
        if (!fl) return;
        collide(f, true, pr, [&](int d, C post) {
            store_dev<P>(B, (unsigned)(d * nc + me), d, post, rho_fd);
        });
    };

    if (lists) {
        // workgroup = 256 consecutive listed nodes of one z plane; a plane with more than
        // ntx * 256 listed nodes gives each of its workgroups further chunks, ntx apart
        const int lb = tl % ntx, z = tl / ntx;
        const int cnt = s.ccnt[pz_off + z];
        if (lb * 256 >= cnt) {
            if (s.pzmap[pz_off + z] >= 0 && threadIdx.x == 0) {
                double *o = s.pprt + (long long)g * s.nzt * 4;
                o[0] = 0.0; o[1] = 0.0; o[2] = 0.0; o[3] = 0.0;
            }
            return;
        }
        for (int lbx = lb; lbx * 256 < cnt; lbx += ntx) {
            const int kk = lbx * 256 + (int)threadIdx.x;
            const bool v = kk < cnt;
            const int c = v ? s.clist[cell_off + (long long)z * nxy + kk] - z * nxy : 0;
            // the node's first link word: under compact storage the copy at its slot
            unsigned long long word = kSolidWord;
            if (v) {
                const long long slot = cell_off + (long long)z * nxy + kk;
                if constexpr (CMP) {
                    word = s.lwc[slot];
                    if (full_compact) {
                        word = compact_word(s.lw[cell_off + z * nxy + c]);
                        s.lwc[slot] = word;
                    }
                } else {
                    word = s.lw[cell_off + z * nxy + c];
                }
            }
            const int jj = c / nx;
            const uint2 *lrt = nullptr;
            int jb = 0, nrows = 0;
            if constexpr (CMP) {
                // the chunk's nodes lie in rows jr[0] .. jr[1] (x-fastest list order): stage
                // the row-table words of their source rows once for the workgroup, unless
                // they do not fit (then each thread reads its own from the tables)
                const int last = min(cnt - lbx * 256, 256) - 1;
                if (threadIdx.x == 0) jr[0] = jj;
                if ((int)threadIdx.x == last) jr[1] = jj;
                __syncthreads();
                jb = jr[0] - 1;
                nrows = jr[1] - jr[0] + 3;
                const int tot = 3 * nrows * nw;
                if (tot <= kRtLds) {
                    const uint2 *rtab = s.rt + rt_off;
                    for (int w = threadIdx.x; w < tot; w += 256) {
                        const int pz = w / (nrows * nw), rem = w - pz * (nrows * nw);
                        const int u = rem / nw, wq = rem - u * nw;
                        const int zz = wrapc(z + pz - 1, nz), jg = wrapc(jb + u, ny);
                        const uint2 rw = rtab[((long long)zz * ny + jg) * nw + wq];
                        rt_lds[w] = make_uint2(rw.x, rw.y + (unsigned)(zz * nxy));
                    }
                    lrt = rt_lds;
                }
                __syncthreads();
            }
            double pr[4] = {0.0, 0.0, 0.0, 0.0};
            const int i = c - jj * nx;
            bool general = true;
            if constexpr (CMP && sizeof(S) == 2) {
                const bool edge = (i == 0 && bc0 != 0) || (i == nx - 1 && bc1 != 0) || (jj == 0 && bc2 != 0) ||
                                  (jj == ny - 1 && bc3 != 0);
                general = !lrt || (z == 0 && bc4 != 0) || (z == nz - 1 && bc5 != 0) || __ballot(v && edge) != 0ull;
                // (a lane past the plane's list takes the slot of the workgroup's first node)
                if (!general)
                    compact_node(i, v ? jj : jb + 1, z, z * nxy + (v ? kk : lbx * 256), v, lrt, jb, nrows, word, pr);
            }
            if (general) node(i, jj, z, z * nxy + kk, v, lrt, jb, nrows, word, pr);
            probes(z, 0, lbx != lb, pr);
            // (the next chunk stages its own rows once every thread is done with these)
            if constexpr (CMP) __syncthreads();
        }
    } else {
        const int bxl = uni(M->bx_log2);
        const int lx = threadIdx.x & ((1 << bxl) - 1), ly = threadIdx.x >> bxl;
        const int tx = tl % ntx, trem = tl / ntx, ty = trem % nty, tz = trem / nty;
        const int i = (tx << bxl) + lx;
        const int j = ty * uni(M->by) + ly;
        const int z0 = tz * s.nzt, z1 = min(z0 + s.nzt, nz);
        const bool vij = (i < nx) && (j < ny);
        // Away from walls, density faces, particles and solid nodes a node pulls each direction
        // from a fixed offset: nine offsets within a plane per column, the planes' and the
        // directions' offsets in scalar registers.  A wave whose nodes are all of that kind
        // takes this path, about half the vector instructions of the general one, which bound
        // the 16-bit storage (pure fluid 96 x 96 x 384, us per launch: BF16 112 -> 64,
        // FP16 84 -> 66, FP32 117 -> 109 of 105 at the rate of a device copy).
        const bool edge = (i == 0 && bc0 != 0) || (i == nx - 1 && bc1 != 0) || (j == 0 && bc2 != 0) ||
                          (j == ny - 1 && bc3 != 0);
        for (int z = z0; z < z1; ++z) {
            double pr[4] = {0.0, 0.0, 0.0, 0.0};
            // (a set without particles has no link words to read)
            unsigned long long word = 0ull;
            if (s.ptot > 0 && vij) word = s.lw[cell_off + (z * ny + j) * nx + i];
            const bool face = (z == 0 && bc4 != 0) || (z == nz - 1 && bc5 != 0);
            if (face || __ballot(vij && (edge || word != 0ull)) != 0ull) {
                node(i, j, z, 0, vij, nullptr, 0, 0, word, pr);
            } else if (vij) {
                const int zs[3] = {z > 0 ? z - 1 : nz - 1, z, z < nz - 1 ? z + 1 : 0};
                // (recomputed per plane: kept across the general path they would spill)
                int ic = i, jc = j;
                asm volatile("" : "+v"(ic), "+v"(jc));
                const int xs[3] = {ic > 0 ? ic - 1 : nx - 1, ic, ic < nx - 1 ? ic + 1 : 0};
                const int ys[3] = {jc > 0 ? jc - 1 : ny - 1, jc, jc < ny - 1 ? jc + 1 : 0};
                unsigned vo[9]; // source (x - c_x, y - c_y) at [3 (1 - c_y) + 1 - c_x]
#pragma unroll
                for (int q = 0; q < 9; ++q) vo[q] = (unsigned)(ys[q / 3] * nx + xs[q % 3]);
                C f[kQ];
                S raw[kQ];
#pragma unroll
                for (int e = 0; e < kQ; ++e)
                    raw[e] = ldo(A + ((long long)e * nc + (long long)zs[1 - kCZ[e]] * nxy), vo[3 * (1 - kCY[e]) + 1 - kCX[e]]);
#pragma unroll
                for (int e = 0; e < kQ; ++e) f[e] = decode_dev<P>(raw[e], e, rho_fd);
                collide(f, true, pr, [&](int d, C post) {
                    store_dev<P>(B + ((long long)d * nc + (long long)z * nxy), vo[4], d, post, rho_fd);
                });
            }
            probes(z, z - z0, false, pr);
        }
        // (a set without particles runs no refresh: the re-projection kernel of this step, which
        // advances the step counter, reads the step from here.  At the end of the kernel: after
        // a store the compiler reads the lattice's constants with vector loads, which cost the
        // FCC wave case 4 of 43 us)
        if (s.ptot == 0 && blockIdx.x == 0 && threadIdx.x == 0) *s.tcopy = t;
    }
}

// ---------------------------------------------------------------------------
// particle kernel: links, contacts, motion
// ---------------------------------------------------------------------------

// Node range [lo, lo + ext) along one axis covering [c - h, c + h]: clipped on a bounded
// axis, at most one full period on a periodic one.
__device__ __forceinline__ void axis_range(double c, double h, int n, int per, int &lo, int &ext)
{
    int l = (int)floor(c - h), u = (int)ceil(c + h);
    if (!per) { l = max(l, 0); u = min(u, n - 1); }
    else if (u - l + 1 > n) { l = 0; u = n - 1; }
    lo = l;
    ext = max(u - l + 1, 0);
}


// n / d for 0 <= n < 2^31 and a divisor d > 0 that every lane shares, through the FP64
// reciprocal (rounded within one unit of the quotient, then corrected)
__device__ __forceinline__ int div_uni(int n, int d, double inv)
{
    int q = (int)((double)n * inv);
    const int r = n - q * d;
    if (r < 0) q -= 1;
    else if (r >= d) q += 1;
    return q;
}

constexpr int kLinkScan = 2;     // candidate cells per lane per scan round of a rebuilt chunk
constexpr int kLinkLds = 320;    // entries of a rebuilt chunk kept in LDS for its link-set sums
constexpr int kCellLds = kLinkLds; // candidate cells of a rebuilt chunk listed at a time

// Direction masks over the links e (d = e*, c_d = -c_e), for sums over a node's links by
// counting: per axis and weight class (w = 1/18 on the axes, e < 6; 1/36 on the
// diagonals) the links whose c_d component is +1 or -1 ...
constexpr unsigned link_mask(int axis, int sign, bool diag)
{
    unsigned m = 0u;
    for (int e = 0; e < kQ - 1; ++e) {
        const int c = -(axis == 0 ? kCX[e] : axis == 1 ? kCY[e] : kCZ[e]);
        if (c == sign && (e >= 6) == diag) m |= 1u << e;
    }
    return m;
}
// ... and the diagonal links whose components along axes a and b have the product +1 or -1
constexpr unsigned pair_mask(int a, int b, int sign)
{
    unsigned m = 0u;
    for (int e = 6; e < kQ - 1; ++e) {
        const int ca = a == 0 ? kCX[e] : a == 1 ? kCY[e] : kCZ[e];
        const int cb = b == 0 ? kCX[e] : b == 1 ? kCY[e] : kCZ[e];
        if (ca * cb == sign) m |= 1u << e;
    }
    return m;
}

// Rows of nodes around a centre: the two intervals of x (unwrapped, relative to the integer
// base) whose distance from the centre lies between the radii of inner2 and outer2 (squared;
// inner2 <= 0: one interval), for a row at squared distance rho2 from the axis through the
// centre; fx is the centre's x relative to the base.  FP32, widened by eps: a superset, whose
// nodes are then tested exactly.
struct RowSpan { int a0, a1, b0, b1; };
__device__ __forceinline__ RowSpan row_span(float rho2, float fx, float inner2, float outer2)
{
    constexpr float eps = 1e-4f;
    RowSpan r = {0, -1, 0, -1};
    const float h2 = outer2 - rho2;
    if (h2 < 0.0f) return r;
    const float h = sqrtf(h2) + eps;
    const float l2 = inner2 - rho2;
    const int lo = (int)ceilf(fx - h), hi = (int)floorf(fx + h);
    if (l2 <= 0.0f) {
        r.a0 = lo; r.a1 = hi;
        return r;
    }
    const float l = sqrtf(l2) - eps;
    const int ml = (int)floorf(fx - l), mr = (int)ceilf(fx + l);
    r.a0 = lo; r.a1 = ml;
    r.b0 = max(mr, ml + 1); r.b1 = hi;
    return r;
}

// Node range [lo, hi] of one axis (unwrapped) within h of c: clipped on a bounded axis, at
// most one period, centred on c, on a periodic one.
__device__ __forceinline__ void near_range(double c, double h, int n, int per, int &lo, int &hi)
{
    lo = (int)ceil(c - h);
    hi = (int)floor(c + h);
    if (per) {
        if (hi - lo + 1 > n) {
            lo = (int)ceil(c - 0.5 * (double)n);
            hi = lo + n - 1;
        }
    } else {
        lo = max(lo, 0);
        hi = min(hi, n - 1);
    }
}

// Margin of the FP32 row tests for spheres of radius R: rounding of squared distances, of
// order R^2 2^-23, shifts a radius by about R 2^-23.
__device__ __forceinline__ double row_margin(double R) { return 2e-5 + 1e-6 * R; }

// Rebuild of one chunk of a particle's link entries, the nodes with links of p in a z-slab
// around it (by the wave of the calling lanes): needed when the slabs were laid out anew, the
// node lists were rebuilt (storage slots move) or a link word of the slab changed in the
// previous step; every other chunk keeps its entries.  The candidates are the nodes with R <
// |x - X| <= R + sqrt(2) (a link's source lies inside p), found row by row from the sphere's
// equation, so the rebuild loads only their link words: one round of loads for the usual
// chunk (about 190 candidates at R = 8.5), then the slots of the nodes that have links.
// Returns the number of entries.
template <bool NR>
__device__ __forceinline__ int rebuild_chunk(const DevSet &s, const MemberDev *M, int p, int chunk, int chunks,
                                              double X0, double X1, double X2, int *cells, int2 *segs, int *lc, unsigned *lg, double *zl)
{
    const int lane = threadIdx.x & 63;
    const int pl = p - uni(M->p_off);
    const int nx = uni(M->nx), ny = uni(M->ny), nz = uni(M->nz);
    const int per0 = uni(M->per[0]), per1 = uni(M->per[1]), per2 = uni(M->per[2]);
    const double box0 = uni(M->box[0]), box1 = uni(M->box[1]), box2 = uni(M->box[2]);
    const long long cell_off = uni(M->cell_off);
    const double rho_f = uni(M->rho_f);
    const int nxy = nx * ny;
    const long long lbase = ((long long)p * chunks + chunk) * s.xcap;
    int *xc = s.xcell + lbase;
    int *xs = s.xslot + lbase;
    unsigned *xg = s.xgrp + lbase;
    const double R0 = s.Xref[3 * p], R1 = s.Xref[3 * p + 1], R2 = s.Xref[3 * p + 2];
    const double inv_nxy = 1.0 / (double)nxy, inv_nx = 1.0 / (double)nx;

    // Link-set sums of a rebuilt chunk (the 6 x 6 matrix Z of the implicit update is
    // assembled from them): with S_n = sum over a node's links of 6 w_d rho_f c_d c_d^T and
    // xr its position relative to X_ref, S = sum S_n, Qx = sum [xr] S_n, Wx = sum [xr] S_n
    // [xr]^T ([v] the matrix of v x .).  On a lattice without narrow periodic axes they are
    // summed exactly, in integers, while the chunk's entries are found: S_n = z36 S'_n with
    // S'_n integer (6 w_d rho_f is 2 z36 on the axes and z36 on the diagonals), and xr = I -
    // fr with I the node's integer offset from floor(X_ref) (minimum image) and fr = X_ref -
    // floor(X_ref), so S = z36 sum S', Qx = z36 (sum [I] S' - [fr] sum S') and Wx = z36 (sum
    // [I] S' [I]^T - T - T^T + [fr] (sum S') [fr]^T), T = (sum [I] S') [fr]^T.  (|I| stays
    // below R + 3: the sums of S' and [I] S' fit 32 bits, those of [I] S' [I]^T take 64.)
    const int fl0 = (int)floor(R0), fl1 = (int)floor(R1), fl2 = (int)floor(R2);
    int zsi[15];
    long long zwl[6];
#pragma unroll
    for (int c = 0; c < 15; ++c) zsi[c] = 0;
#pragma unroll
    for (int c = 0; c < 6; ++c) zwl[c] = 0;
    auto add_link_set = [&](int cell, unsigned g) {
        const int kk = div_uni(cell, nxy, inv_nxy), rem = cell - kk * nxy;
        const int jj = div_uni(rem, nx, inv_nx), ii = rem - jj * nx;
        auto arm = [](int c, double R, int fl, int per, double box) {
            const double dx = (double)c - R;
            const int n = (int)box;
            return (c - fl) + ((per && dx > 0.5 * box) ? -n : ((per && dx < -0.5 * box) ? n : 0));
        };
        const int I0 = arm(ii, R0, fl0, per0, box0), I1 = arm(jj, R1, fl1, per1, box1), I2 = arm(kk, R2, fl2, per2, box2);
        auto diag = [&](int axis) {
            return 2 * (int)__popc(g & (link_mask(axis, 1, false) | link_mask(axis, -1, false))) +
                   (int)__popc(g & (link_mask(axis, 1, true) | link_mask(axis, -1, true)));
        };
        auto offd = [&](int a, int b2) {
            return (int)__popc(g & pair_mask(a, b2, 1)) - (int)__popc(g & pair_mask(a, b2, -1));
        };
        const int Sxx = diag(0), Syy = diag(1), Szz = diag(2);
        const int Sxy = offd(0, 1), Sxz = offd(0, 2), Syz = offd(1, 2);
        // [I] S' by columns (column n of S' is (S'_xn, S'_yn, S'_zn)), then row a of
        // [I] S' [I]^T as I x (row a of [I] S')
        // (24-bit multiplies: every factor is far below 2^23)
        auto cross = [](int a0, int a1, int a2, int b0, int b1, int b2, int &c0, int &c1, int &c2) {
            c0 = __mul24(a1, b2) - __mul24(a2, b1);
            c1 = __mul24(a2, b0) - __mul24(a0, b2);
            c2 = __mul24(a0, b1) - __mul24(a1, b0);
        };
        int q00, q10, q20, q01, q11, q21, q02, q12, q22;
        cross(I0, I1, I2, Sxx, Sxy, Sxz, q00, q10, q20);
        cross(I0, I1, I2, Sxy, Syy, Syz, q01, q11, q21);
        cross(I0, I1, I2, Sxz, Syz, Szz, q02, q12, q22);
        zsi[0] += Sxx; zsi[1] += Sxy; zsi[2] += Sxz; zsi[3] += Syy; zsi[4] += Syz; zsi[5] += Szz;
        zsi[6] += q00; zsi[7] += q01; zsi[8] += q02;
        zsi[9] += q10; zsi[10] += q11; zsi[11] += q12;
        zsi[12] += q20; zsi[13] += q21; zsi[14] += q22;
        int w00, w01, w02, w10, w11, w12, w20, w21, w22;
        cross(I0, I1, I2, q00, q01, q02, w00, w01, w02);
        cross(I0, I1, I2, q10, q11, q12, w10, w11, w12);
        cross(I0, I1, I2, q20, q21, q22, w20, w21, w22);
        (void)w10; (void)w20; (void)w21;
        zwl[0] += w00; zwl[1] += w01; zwl[2] += w02; zwl[3] += w11; zwl[4] += w12; zwl[5] += w22;
    };

    // (1) the chunk's candidates in (z, y, x) order, kCellLds at a time, and of them the
    // nodes that hold links of p
    int cntx = 0;
    const double R = s.R[p], mrg = row_margin(R);
    const double reach = R + 1.4142135623730951 + mrg, skip = R - mrg;
    const float inner2 = skip > 0.0 ? (float)(skip * skip) : -1.0f, outer2 = (float)(reach * reach);
    int y0, y1, x0, x1;
    near_range(X0, reach, nx, per0, x0, x1);
    near_range(X1, reach, ny, per1, y0, y1);
    const int ix = (int)floor(X0);
    const float fx = (float)(X0 - (double)ix);
    // the slab's planes, unwrapped next to X_ref (at most one period, or the bounded extent)
    const int zr0 = s.lzr[2 * p], hz = s.lzr[2 * p + 1];
    const int zs = per2 ? zr0 + chunk * hz : max(zr0 + chunk * hz, 0);
    const int ze = min(zr0 + (chunk + 1) * hz, per2 ? zr0 + nz : nz);
    const int nj = max(y1 - y0 + 1, 0), nrow = nj * max(ze - zs, 0);
    const double inv_nj = 1.0 / (double)max(nj, 1);
    for (int row0 = 0; row0 < nrow; row0 += 128) {
        // two consecutive rows per lane (a usual slab has about 70)
        RowSpan sp[2];
        int base_cell[2], na[2], nb[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = row0 + 2 * lane + h;
            sp[h] = {0, -1, 0, -1};
            base_cell[h] = 0;
            if (row < nrow) {
                const int kz = div_uni(row, nj, inv_nj), ky = row - kz * nj;
                int zz = zs + kz, yy = y0 + ky;
                const double dy = (double)yy - X1;
                if (per2) zz = ((zz % nz) + nz) % nz;
                if (per1) yy = yy < 0 ? yy + ny : (yy >= ny ? yy - ny : yy);
                const double dz = mimg((double)zz - X2, per2, box2);
                sp[h] = row_span((float)(dy * dy + dz * dz), fx, inner2, outer2);
                sp[h].a0 = max(sp[h].a0, x0 - ix); sp[h].b0 = max(sp[h].b0, x0 - ix);
                sp[h].a1 = min(sp[h].a1, x1 - ix); sp[h].b1 = min(sp[h].b1, x1 - ix);
                base_cell[h] = zz * nxy + yy * nx;
            }
            na[h] = max(sp[h].a1 - sp[h].a0 + 1, 0);
            nb[h] = max(sp[h].b1 - sp[h].b0 + 1, 0);
        }
        const int own_n = na[0] + nb[0] + na[1] + nb[1];
        int inc = own_n;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        const int total = __builtin_amdgcn_readlane(inc, 63);
        // the lane's four runs of nodes: where each starts in the list, its cell and first x
        {
            int at = inc - own_n;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                segs[4 * lane + 2 * h] = make_int2(base_cell[h], ix + sp[h].a0 - at);
                segs[4 * lane + 2 * h + 1] = make_int2(base_cell[h], ix + sp[h].b0 - (at + na[h]));
                at += na[h] + nb[h];
            }
        }
        for (int part = 0; part < total; part += kCellLds) {
        const int npart = min(total - part, kCellLds);
        // a mark at the first node of each run; a running maximum of the marks then gives each
        // lane its node's run (the lanes writing out their runs node by node took 10 us)
        for (int k = lane; k < npart; k += 64) cells[k] = 0;
        wave_fence();
        {
            int at = inc - own_n - part;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (na[h] > 0 && at + na[h] > 0 && at < npart) cells[max(at, 0)] = 4 * lane + 2 * h + 1;
                at += na[h];
                if (nb[h] > 0 && at + nb[h] > 0 && at < npart) cells[max(at, 0)] = 4 * lane + 2 * h + 2;
                at += nb[h];
            }
        }
        wave_fence();
        int run = 0;
        // kLinkScan cells per lane and round, their link words loaded together; the cells are
        // then taken in list order
        for (int base = 0; base < npart; base += 64 * kLinkScan) {
            unsigned mk[kLinkScan];
            int cl[kLinkScan];
#pragma unroll
            for (int b = 0; b < kLinkScan; ++b) {
                const int k = base + b * 64 + lane;
                mk[b] = k < npart ? 1u : 0u;
                int v = cells[min(k, npart - 1)];
                v = max(v, dpp_i<0x111, 0xF>(v, 0)); // row_shr 1, 2, 4, 8: maxima within rows of 16
                v = max(v, dpp_i<0x112, 0xF>(v, 0));
                v = max(v, dpp_i<0x114, 0xF>(v, 0));
                v = max(v, dpp_i<0x118, 0xF>(v, 0));
                v = max(v, dpp_i<0x142, 0xA>(v, 0)); // row_bcast 15, 31: carried over the rows
                v = max(v, dpp_i<0x143, 0xC>(v, 0));
                v = max(v, run);
                run = __builtin_amdgcn_readlane(v, 63);
                const int2 sg = segs[v - 1];
                int x = sg.y + part + min(k, npart - 1);
                if (per0) x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
                cl[b] = sg.x + x;
            }
            unsigned long long w0b[kLinkScan];
#pragma unroll
            for (int b = 0; b < kLinkScan; ++b) {
                const unsigned long long wr = s.lw[cell_off + cl[b]];
                w0b[b] = mk[b] != 0u ? wr : 0ull;
            }
#pragma unroll
            for (int b = 0; b < kLinkScan; ++b) {
                const int cell = cl[b];
                const unsigned long long w0 = ((unsigned)w0b[b] & 0x3ffffu) != 0u ? w0b[b] : 0ull;
                const unsigned long long w1 = (w0 >> 62) ? s.lw[s.ncell_total + cell_off + cell] : 0ull;
                const int ng = (w0 >> 62) ? 4 : 2;
                // one entry per slot of p at the node: one pass, or more in a set with a
                // narrow lattice, where a node can hold links into two images of p (one slot
                // each)
                int g0 = 0;
                for (int pass = 0; pass < (NR ? 4 : 1); ++pass) {
                    unsigned grp = 0u;
                    int slot = 0;
                    for (int g = g0; g < ng; ++g) {
                        int q;
                        const unsigned gd = slot_dirs(w0, w1, g, q);
                        if (gd != 0u && q == pl) { grp = gd; slot = g; break; }
                    }
                    const bool has = grp != 0u;
                    const unsigned long long bal = __ballot(has);
                    if (bal == 0ull) break;
                    if (has) {
                        const int at = cntx + __popcll(bal & ((1ull << lane) - 1ull));
                        if (at < s.xcap) {
                            xc[at] = cell;
                            xg[at] = grp;
                            // (the first kLinkLds entries also in this wave's LDS, where the
                            // link-set sums read them)
                            if (at < kLinkLds) {
                                lc[at] = cell;
                                lg[at] = grp;
                            }
                        } else {
                            atomicOr(s.flags, 0x40u);
                        }
                        g0 = slot + 1;
                    } else {
                        g0 = ng;
                    }
                    cntx = min(cntx + __popcll(bal), s.xcap);
                }
            }
        }
        wave_fence(); // (the next part marks the list again once every lane has read it)
        }
    }
    {
        if (lane == 0) s.xcnt[p * chunks + chunk] = cntx;
        // (the link-set sums read the entries back, from LDS, or from memory for a chunk
        // with more than kLinkLds entries: the wave's writes are made visible to the wave
        // itself; the other waves of its workgroup rebuild other chunks)
        if (cntx <= kLinkLds) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
    }
    const bool from_lds = cntx <= kLinkLds;
    // storage slots of the entries' nodes (kept in LDS too, over the candidates), four a lane
    // in flight
    for (int base = 0; base < cntx; base += 256) {
        int cell[4], ns[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int k = min(base + 64 * b + lane, cntx - 1);
            cell[b] = from_lds ? lc[k] : xc[k];
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int kk = div_uni(cell[b], nxy, inv_nxy), rem = cell[b] - kk * nxy;
            const int jj = div_uni(rem, nx, inv_nx);
            ns[b] = node_slot(s, M, cell[b], rem - jj * nx, jj, kk);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int k = base + 64 * b + lane;
            if (k >= cntx) continue;
            xs[k] = ns[b];
            if (from_lds) cells[k] = ns[b];
        }
    }

    // Positions of the entries' nodes relative to the particle's reference point X_ref, as in
    // the link pass.
    const double z18 = rho_f / 3.0, z36 = rho_f / 6.0;                  // 6 rho_f w_d
    // (in a set with a narrow lattice the entry's image of p is the one that holds its link
    // group: its arm from the current centre X, as group_arm, plus the small displacement
    // X - X_ref)
    const double dX0 = mimg(X0 - R0, per0, box0), dX1 = mimg(X1 - R1, per1, box1), dX2 = mimg(X2 - R2, per2, box2);
    auto rel_pos = [&](int cell, unsigned g, double &x0, double &x1, double &x2) {
        const int kk = div_uni(cell, nxy, inv_nxy), rem = cell - kk * nxy;
        const int jj = div_uni(rem, nx, inv_nx), ii = rem - jj * nx;
        if constexpr (NR) {
            group_arm<true>(M, g, ii, jj, kk, X0, X1, X2, x0, x1, x2);
            x0 += dX0; x1 += dX1; x2 += dX2;
        } else {
            x0 = mimg((double)ii - R0, per0, box0);
            x1 = mimg((double)jj - R1, per1, box1);
            x2 = mimg((double)kk - R2, per2, box2);
        }
    };

    // (2) link-set sums of a rebuilt chunk: S, Qx, Wx (21 values, cached per chunk); exact
    // integer sums from the scan, or, in a set with a narrow lattice, FP64 sums over the
    // entries in list order
    if (!NR) {
        if (from_lds)
            for (int k = lane; k < cntx; k += 64) add_link_set(lc[k], lg[k]);
        else
            for (int k = lane; k < cntx; k += 64) add_link_set(xc[k], xg[k]);
        int si[15];
#pragma unroll
        for (int c = 0; c < 15; ++c) si[c] = wave_sum_i(zsi[c]);
        double wl[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) wl[c] = wave_sum((double)zwl[c]); // exact: integers below 2^53
        if (lane == 0) {
            const double f0 = R0 - (double)fl0, f1 = R1 - (double)fl1, f2 = R2 - (double)fl2;
            double Ss[3][3], Qs[3][3], Ws[3][3];
            {
                int z = 0;
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int c = a; c < 3; ++c) { Ss[a][c] = (double)si[z]; Ss[c][a] = (double)si[z]; ++z; }
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int c = 0; c < 3; ++c) Qs[a][c] = (double)si[z++];
                z = 0;
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int c = a; c < 3; ++c) { Ws[a][c] = wl[z]; Ws[c][a] = wl[z]; ++z; }
            }
            // fr x (column n of M) for M = sum S'; fr x (row a of M) for M = sum [I] S' and
            // for M = [fr] sum S'
            double FS[3][3], T[3][3], FSF[3][3];
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                FS[0][n] = f1 * Ss[2][n] - f2 * Ss[1][n];
                FS[1][n] = f2 * Ss[0][n] - f0 * Ss[2][n];
                FS[2][n] = f0 * Ss[1][n] - f1 * Ss[0][n];
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                T[a][0] = f1 * Qs[a][2] - f2 * Qs[a][1];
                T[a][1] = f2 * Qs[a][0] - f0 * Qs[a][2];
                T[a][2] = f0 * Qs[a][1] - f1 * Qs[a][0];
                FSF[a][0] = f1 * FS[a][2] - f2 * FS[a][1];
                FSF[a][1] = f2 * FS[a][0] - f0 * FS[a][2];
                FSF[a][2] = f0 * FS[a][1] - f1 * FS[a][0];
            }
            double *zc = s.zcache + ((long long)p * chunks + chunk) * kZComp;
            int z = 0;
            auto put = [&](double v) { zc[z] = v; if (zl) zl[z] = v; ++z; };
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int c = a; c < 3; ++c) put(z36 * Ss[a][c]);
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int c = 0; c < 3; ++c) put(z36 * (Qs[a][c] - FS[a][c]));
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int c = a; c < 3; ++c) put(z36 * (((Ws[a][c] - T[a][c]) - T[c][a]) + FSF[a][c]));
        }
    }
    if (NR) {
        double zs[21];
#pragma unroll
        for (int c = 0; c < 21; ++c) zs[c] = 0.0;
        for (int k = lane; k < cntx; k += 64) {
            const unsigned g = from_lds ? lg[k] : xg[k];
            double x0, x1, x2;
            rel_pos(from_lds ? lc[k] : xc[k], g, x0, x1, x2);
            // S_n = sum 6 w_d rho_f c_d c_d^T over the node's links, from counts
            auto diag = [&](int axis) {
                return z18 * (double)__popc(g & (link_mask(axis, 1, false) | link_mask(axis, -1, false))) +
                       z36 * (double)__popc(g & (link_mask(axis, 1, true) | link_mask(axis, -1, true)));
            };
            auto offd = [&](int a, int b2) {
                // (the counts are unsigned: take the difference as a signed integer)
                const int n = (int)__popc(g & pair_mask(a, b2, 1)) - (int)__popc(g & pair_mask(a, b2, -1));
                return z36 * (double)n;
            };
            const double Sxy = offd(0, 1), Sxz = offd(0, 2), Syz = offd(1, 2);
            const double Sm[3][3] = {{diag(0), Sxy, Sxz}, {Sxy, diag(1), Syz}, {Sxz, Syz, diag(2)}};
            // Q = [xr] S_n (row a: xr x (column of S_n)), W = Q [xr]^T
            double Qm[3][3], Wm[3][3];
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                Qm[0][n] = x1 * Sm[2][n] - x2 * Sm[1][n];
                Qm[1][n] = x2 * Sm[0][n] - x0 * Sm[2][n];
                Qm[2][n] = x0 * Sm[1][n] - x1 * Sm[0][n];
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                Wm[a][0] = x1 * Qm[a][2] - x2 * Qm[a][1];
                Wm[a][1] = x2 * Qm[a][0] - x0 * Qm[a][2];
                Wm[a][2] = x0 * Qm[a][1] - x1 * Qm[a][0];
            }
            int z = 0;
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b2 = a; b2 < 3; ++b2) zs[z++] += Sm[a][b2];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b2 = 0; b2 < 3; ++b2) zs[z++] += Qm[a][b2];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b2 = a; b2 < 3; ++b2) zs[z++] += Wm[a][b2];
        }
#pragma unroll
        for (int c = 0; c < 21; ++c) zs[c] = wave_sum(zs[c]);
        if (lane == 0) {
            double *zc = s.zcache + ((long long)p * chunks + chunk) * kZComp;
#pragma unroll
            for (int c = 0; c < 21; ++c) { zc[c] = zs[c]; if (zl) zl[c] = zs[c]; }
        }
    }
    return cntx;
}

// ---------------------------------------------------------------------------
// motion: contacts and the implicit update of a particle, by one wave
// ---------------------------------------------------------------------------

// Hertz / Mindlin contacts (Eqs. fdLawn, fdLaws) of particle p with the particles of its near
// list at X(t), V(t), summed over the wave (lane c < 6 returns component c of force and
// torque; mode 0), with the contact histories of the next step; or the near-list build: every particle within R_p + R_q +
// kNearMargin (mode 1).
__device__ __forceinline__ double contact_pass(const DevSet &s, const MemberDev *M, int p, int par, int mode)
{
    const int lane = threadIdx.x & 63;
    const double *Xo = s.X[par], *Vo = s.V[par], *Wo = s.W[par];
    const double X0 = Xo[3 * p], X1 = Xo[3 * p + 1], X2 = Xo[3 * p + 2];
    const double R = s.R[p];
    const int nn_ld = s.nnear[p];
    const int nl_ld = s.nearl[(long long)p * kNearCap + (lane & (kNearCap - 1))];
    const int hno = s.hn[par][p];
    const int per0 = M->per[0], per1 = M->per[1], per2 = M->per[2];
    const double box0 = M->box[0], box1 = M->box[1], box2 = M->box[2];

    // contacts over the near list (mode 0) or the near-list build (mode 1)
    const int q0 = M->p_off, nq = M->np;
    const double E = M->E, nu = M->nu, mu = M->mu;
    const int *hjo = s.hj[par] + (long long)p * kHistCap;
    const double *hfo = s.hf[par] + (long long)p * kHistCap * 3;
    int *hjn = s.hj[par ^ 1] + (long long)p * kHistCap;
    double *hfn = s.hf[par ^ 1] + (long long)p * kHistCap * 3;
    double con[6] = {0, 0, 0, 0, 0, 0};
    int near_total = 0, hist_total = 0;
    const bool build = mode != 0;
    const int ncand = build ? nq : min(nn_ld, kNearCap);
    const unsigned long long below = (1ull << lane) - 1ull;
    static_assert(kNearCap <= 64, "a near list fits one wave");
    for (int base = 0; base < ncand; base += 64) {
        const int jj = base + lane;
        // (a near list has at most kNearCap <= 64 entries: lane jj < ncand took entry jj)
        const int q = (jj < ncand) ? (build ? q0 + jj : nl_ld) : -1;
        bool isnear = false, keep = false;
        double ftn[3] = {0, 0, 0};
        if (jj < ncand && q != p) {
            const double Y0 = Xo[3 * q], Y1 = Xo[3 * q + 1], Y2 = Xo[3 * q + 2], Rq = s.R[q];
            const double d0 = mimg(Y0 - X0, per0, box0);
            const double d1 = mimg(Y1 - X1, per1, box1);
            const double d2 = mimg(Y2 - X2, per2, box2);
            const double dist = sqrt((d0 * d0 + d1 * d1) + d2 * d2);
            isnear = dist <= R + Rq + kNearMargin;
            const double un = R + Rq - dist;
            if (mode == 0 && un > 0.0) {
                // Eq. (fdLawn): Hertz normal force, pushing p away from q
                const double n0 = d0 / dist, n1 = d1 / dist, n2 = d2 / dist;
                const double rstar = 1.0 / (1.0 / R + 1.0 / Rq);
                const double fn = 2.0 * E * un * sqrt(rstar * un) / (3.0 * (1.0 - nu * nu));
                con[0] += -fn * n0; con[1] += -fn * n1; con[2] += -fn * n2;
                if (mu > 0.0) {
                    // Eq. (fdLaws): incremental Mindlin spring, Coulomb cap
                    double fo[3] = {0, 0, 0};
                    for (int h = 0; h < hno; ++h)
                        if (hjo[h] == q) { fo[0] = hfo[3 * h]; fo[1] = hfo[3 * h + 1]; fo[2] = hfo[3 * h + 2]; }
                    const double a0 = (R - 0.5 * un) * n0, a1 = (R - 0.5 * un) * n1, a2 = (R - 0.5 * un) * n2;
                    const double b0 = -(Rq - 0.5 * un) * n0, b1 = -(Rq - 0.5 * un) * n1, b2 = -(Rq - 0.5 * un) * n2;
                    const double *Vq = Vo + 3 * q, *Wq = Wo + 3 * q, *Vp = Vo + 3 * p, *Wp = Wo + 3 * p;
                    const double wa0 = Wp[1] * a2 - Wp[2] * a1, wa1 = Wp[2] * a0 - Wp[0] * a2, wa2 = Wp[0] * a1 - Wp[1] * a0;
                    const double wb0 = Wq[1] * b2 - Wq[2] * b1, wb1 = Wq[2] * b0 - Wq[0] * b2, wb2 = Wq[0] * b1 - Wq[1] * b0;
                    const double v0 = (Vp[0] + wa0) - (Vq[0] + wb0);
                    const double v1 = (Vp[1] + wa1) - (Vq[1] + wb1);
                    const double v2 = (Vp[2] + wa2) - (Vq[2] + wb2);
                    const double vn = v0 * n0 + v1 * n1 + v2 * n2;
                    const double fon = fo[0] * n0 + fo[1] * n1 + fo[2] * n2;
                    const double kt = 2.0 * E * sqrt(rstar * un) / ((1.0 + nu) * (2.0 - nu));
                    ftn[0] = (fo[0] - fon * n0) - kt * (v0 - vn * n0);
                    ftn[1] = (fo[1] - fon * n1) - kt * (v1 - vn * n1);
                    ftn[2] = (fo[2] - fon * n2) - kt * (v2 - vn * n2);
                    const double fm = sqrt(ftn[0] * ftn[0] + ftn[1] * ftn[1] + ftn[2] * ftn[2]);
                    if (fm > mu * fn) { const double sc = mu * fn / fm; ftn[0] *= sc; ftn[1] *= sc; ftn[2] *= sc; }
                    con[0] += ftn[0]; con[1] += ftn[1]; con[2] += ftn[2];
                    con[3] += a1 * ftn[2] - a2 * ftn[1];
                    con[4] += a2 * ftn[0] - a0 * ftn[2];
                    con[5] += a0 * ftn[1] - a1 * ftn[0];
                    keep = true;
                }
            }
        }
        if (build) {
            const unsigned long long bal = __ballot(isnear);
            if (isnear) {
                const int slot = near_total + __popcll(bal & below);
                if (slot < kNearCap) s.nearl[(long long)p * kNearCap + slot] = q;
                else atomicOr(s.flags, 0x2u);
            }
            near_total += __popcll(bal);
        }
        if (mode == 0 && mu > 0.0) {
            const unsigned long long bal = __ballot(keep);
            if (keep) {
                const int slot = hist_total + __popcll(bal & below);
                if (slot < kHistCap) {
                    hjn[slot] = q;
                    hfn[3 * slot] = ftn[0]; hfn[3 * slot + 1] = ftn[1]; hfn[3 * slot + 2] = ftn[2];
                } else {
                    atomicOr(s.flags, 0x8u);
                }
            }
            hist_total += __popcll(bal);
        }
    }
    if (lane == 0) {
        if (build) {
            s.nnear[p] = min(near_total, kNearCap);
        }
        if (mode == 0) s.hn[par ^ 1][p] = min(hist_total, kHistCap);
    }
    double mine = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        const double v = wave_sum(con[c]);
        mine = lane == c ? v : mine;
    }
    return mine;
}

// The lane's own share of a particle's update: lanes 0..2 the force rows, 3..5 the torque rows
// (loaded before the link sums are known).
struct MotionRow {
    double mi, vel, pend, fg; // mass or inertia, V or Omega, the pending impulse, F_g or nothing
    double X[3], Xr[3];
    int fixed;
};
__device__ __forceinline__ MotionRow motion_row(const DevSet &s, int p, int par)
{
    const int lane = threadIdx.x & 63, a = lane % 3;
    const bool rot = lane >= 3;
    const bool hyd = !s.fluid_off; // (otherwise there are no conversion momenta)
    MotionRow r;
    r.mi = rot ? s.I[p] : s.m[p];
    r.vel = (rot ? s.W[par] : s.V[par])[3 * p + a];
    r.pend = hyd ? (rot ? s.Lh : s.Ph)[3 * p + a] : 0.0;
    r.fg = s.Fg[3 * p + a];
#pragma unroll
    for (int c = 0; c < 3; ++c) { r.X[c] = s.X[par][3 * p + c]; r.Xr[c] = s.Xref[3 * p + c]; }
    r.fixed = s.fixed[p];
    return r;
}

// Eqs. (translate), (rotate) over the step with symplectic Euler, dt = 1: contacts, the external
// force, the conversion impulses of the previous re-projection, and the momentum exchanged
// with the fluid in this step, F0 - Z (V', Omega') from the link sums lp (F0, sum xr x G, S,
// Qx, Wx, in LDS), solved for the velocities of the step, (M + Z)(V', Omega') = M (V, Omega) +
// F0 + the rest; X(t+1) = X(t) + V'.  F_h, T_h of Eqs. (coupleF), (coupleT) are reported.  Fixed
// particles stay.  The fluid kernel's wall state (X(t), V', Omega') is written in FP32.
// Latency-bound: Z is assembled one element per lane (work: 45 values in LDS), the system is
// factored as L D L^T one row per lane, one division per pivot (the motion kernel of the FCC
// wave case with all of it in one lane, 203 registers: 12.0 us, now 8.7).
__device__ __forceinline__ void motion_update(const DevSet &s, const MemberDev *M, int p, int par, long long t,
                                              const MotionRow &row, double con, double *lp, double *work)
{
    const int lane = threadIdx.x & 63;
    double *DS = work, *Z = work + 9;
    const double box[3] = {M->box[0], M->box[1], M->box[2]};
    const int per[3] = {M->per[0], M->per[1], M->per[2]};
    // delta = X - X_ref: the torque arm of a link node is xr - delta
    double dl[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) dl[a] = mimg(row.X[a] - row.Xr[a], per[a], box[a]);
    auto dsel = [&](int a) { return a == 0 ? dl[0] : (a == 1 ? dl[1] : dl[2]); };
    const int a1 = (lane + 1) % 3, a2 = (lane + 2) % 3;
    // T0 = sum xr x G - delta x F0
    double f0 = lp[min(lane, 5)];
    if (lane >= 3) f0 -= dsel(a1) * lp[a2] - dsel(a2) * lp[a1];
    // Z: Z_VV = S, Z_OmegaV = Qx - [delta] S, Z_OmegaOmega = Wx - Qx [delta]^T - [delta] Qx^T
    // + [delta] S [delta]^T, with [delta] v = delta x v; lane 3 a + c takes element (a, c)
    const int l9 = min(lane, 8), ra = l9 / 3, rc = l9 - 3 * ra;
    auto sym = [](int a, int c) { const int lo = min(a, c); return lo * (5 - lo) / 2 + max(a, c); };
    const double *Sp = lp + kLinkComp, *Qp = Sp + 6, *Wp = Qp + 9;
    double Da[3], Dc[3];
    {
        const double v1 = dsel((ra + 1) % 3), v2 = dsel((ra + 2) % 3);
        const double u1 = dsel((rc + 1) % 3), u2 = dsel((rc + 2) % 3);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            Da[k] = k == ra ? 0.0 : (k == (ra + 1) % 3 ? -v2 : v1);
            Dc[k] = k == rc ? 0.0 : (k == (rc + 1) % 3 ? -u2 : u1);
        }
    }
    double ds = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) ds += Da[k] * Sp[sym(k, rc)];
    const double zov = Qp[3 * ra + rc] - ds;
    if (lane < 9) {
        DS[lane] = ds;
        Z[6 * ra + rc] = Sp[sym(ra, rc)];
        Z[6 * rc + 3 + ra] = zov;
        Z[6 * (3 + ra) + rc] = zov;
    }
    wave_fence();
    {
        double qd = 0.0, dq = 0.0, dsd = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            qd += Qp[3 * ra + k] * Dc[k];
            dq += Da[k] * Qp[3 * rc + k];
            dsd += DS[3 * ra + k] * Dc[k];
        }
        const double zoo = ((Wp[sym(ra, rc)] - qd) - dq) + dsd;
        if (lane < 9 && ra <= rc) {
            Z[6 * (3 + ra) + 3 + rc] = zoo;
            Z[6 * (3 + rc) + 3 + ra] = zoo;
        }
    }
    wave_fence();
    // (M + Z)(V', Omega') = M (V, Omega) + F0 + contacts + F_g + pending impulses
    const int i6 = min(lane, 5);
    double r[6], L[6], x[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        r[c] = Z[6 * i6 + c];
        if (c == i6) r[c] += row.mi;
    }
    double b;
    {
        double sum = f0 + row.pend;
        if (lane < 3) sum += row.fg;
        b = row.mi * row.vel + (sum + con);
    }
    double iD = 0.0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const double id = 1.0 / readlane_d(r[j], j);
        if (i6 == j) iD = id;
        L[j] = r[j] * id;
#pragma unroll
        for (int c = j + 1; c < 6; ++c) r[c] -= L[j] * readlane_d(r[j], c);
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const double bk = readlane_d(b, k);
        if (i6 > k) b -= L[k] * bk;
    }
    b *= iD;
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        double v = readlane_d(b, i);
#pragma unroll
        for (int k = i + 1; k < 6; ++k) v -= readlane_d(L[i], k) * x[k];
        x[i] = v;
    }
    if (row.fixed) {
#pragma unroll
        for (int a = 0; a < 6; ++a) x[a] = 0.0;
    } else {
        // a step beyond 0.25 lu (or a non-finite state) is an error (status 0x10); the
        // particle is then held to a step of 0.25 lu and inside the lattice, so that
        // every index derived from its position stays in range
        const double v2 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
        const bool fin = isfinite(v2) && isfinite(x[3]) && isfinite(x[4]) && isfinite(x[5]);
        if (!fin || !(v2 <= 0.0625)) {
            if (lane == 0) atomicOr(s.flags, 0x10u);
            if (!fin) {
#pragma unroll
                for (int a = 0; a < 6; ++a) x[a] = 0.0;
            } else {
                const double sc = 0.25 / sqrt(v2);
#pragma unroll
                for (int a = 0; a < 3; ++a) x[a] *= sc;
            }
        }
    }
    // F_h, T_h: the momentum exchanged with the fluid over the step, F0 - Z (V', Omega'), plus
    // the pending impulses used here (Eqs. coupleF, coupleT)
    double zx = 0.0, xl = x[0];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        zx += Z[6 * i6 + c] * x[c];
        xl = lane == c ? x[c] : xl;
    }
    if (lane < 3) {
        const int a = lane;
        const double bx = a == 0 ? box[0] : (a == 1 ? box[1] : box[2]);
        const int pr = a == 0 ? per[0] : (a == 1 ? per[1] : per[2]);
        const double xc = a == 0 ? row.X[0] : (a == 1 ? row.X[1] : row.X[2]);
        s.Fh[3 * p + a] = (f0 - zx) + row.pend;
        if (s.pv_ring > 0) s.pvring[((t % s.pv_ring) * (long long)s.ptot + p) * 3 + a] = xl;
        s.V[par ^ 1][3 * p + a] = xl;
        double xa = xc + xl;
        if (row.fixed) {
            xa = xc;
        } else if (pr) {
            if (xa >= bx) xa -= bx;
            else if (xa < 0.0) xa += bx;
        } else {
            if (xa < 0.0 || xa > bx - 1.0) atomicOr(s.flags, 0x10u);
            xa = fmin(fmax(xa, 0.0), bx - 1.0);
        }
        s.X[par ^ 1][3 * p + a] = xa;
    } else if (lane < 6) {
        const int a = lane - 3;
        s.Th[3 * p + a] = (f0 - zx) + row.pend;
        s.W[par ^ 1][3 * p + a] = xl;
    }
    // the fluid kernel's wall state of this step: X(t) and the new velocities
    if (lane == 0) pack_state(s.pf[par] + 12 * p, row.X, x, x + 3);
}

// One wave per particle: mode 1, the near list and the FP32 state copy of a set-up (later lists
// are built by the re-projection kernel); mode 0, the step's contacts and motion, unless a wave
// of the link kernel does both.  MANY: more than kChunks chunks a particle (the loop over them
// costs the others 0.2 us a launch).
constexpr int kMotionWaves = 4;
constexpr int kMotionWork = 45;
template <bool MANY>
__global__ __launch_bounds__(64 * kMotionWaves) void k_motion(DevSet s, int mode, int only)
{
    __shared__ double lp[kMotionWaves][kLinkComp + kZComp], work[kMotionWaves][kMotionWork];
    const long long t = *s.tstep;
    const int par = (int)(t & 1);
    const int lane = threadIdx.x & 63, wv = (int)(threadIdx.x >> 6);
    const int p = blockIdx.x * kMotionWaves + wv;
    if (p >= s.ptot) return; // the whole wave: waves never synchronise here
    const int m = s.pmem[p];
    const MotionRow row = motion_row(s, p, par);
    // the link pass's sums (with the hydrodynamics switched off there are none)
    if (mode == 0 && lane < kLinkComp + kZComp) {
        double v = 0.0;
        if (!s.fluid_off) {
            const bool part = lane < kLinkComp;
            const int stride = part ? kLinkComp : kZComp;
            const long long c0 = (long long)p * (MANY ? s.chunks : kChunks);
            const double *pp = part ? s.ppart + c0 * kLinkComp + lane : s.zcache + c0 * kZComp + (lane - kLinkComp);
            double ch[kChunks];
#pragma unroll
            for (int q = 0; q < kChunks; ++q) ch[q] = pp[q * stride];
#pragma unroll
            for (int q = 0; q < kChunks; ++q) v += ch[q];
            if constexpr (MANY)
                for (int q0 = kChunks; q0 < s.chunks; q0 += kChunks) {
#pragma unroll
                    for (int q = 0; q < kChunks; ++q) ch[q] = pp[(q0 + q) * stride];
#pragma unroll
                    for (int q = 0; q < kChunks; ++q) v += ch[q];
                }
        }
        lp[wv][lane] = v;
    }
    const MemberDev *M = s.mem + m;
    if (p - M->p_off >= M->np) return;
    if (only >= 0 && m != only) return;
    const double con = contact_pass(s, M, p, par, mode);
    if (mode != 0) {
        if (lane == 0) pack_state(s.pf[par] + 12 * p, s.X[par] + 3 * p, s.V[par] + 3 * p, s.W[par] + 3 * p);
        return;
    }
    wave_fence();
    motion_update(s, M, p, par, t, row, con, lp[wv], work[wv]);
}

// Link pass, one wave per (particle p, chunk of p's link entries).  A link of p is a fluid
// node x and a direction e whose source x - c_e lies in p; with d = e* pointing into p,
// Eq. (fFS) with Eq. (mem) substituted gives
//   F = c_d f~_d(x,t) - c_e f_e(x,t+1) = 2 c_d f~_d(x,t) - (2 w_d / c_s^2) rho_f c_d (c_d . V_b),
// V_b = V_p + Omega_p x (x_b - X_p), x_b = x + c_d/2.  Since (x_b - X_p) x c_d = (x - X_p) x c_d
// = r x c_d, the force and its torque about X_p over the step are (F, T) = F0 - Z (V, Omega)
// with F0 = (G, r x G), G = sum 2 c_d f~_d(x,t), and Z = sum (2 w_d / c_s^2) rho_f a_d a_d^T,
// a_d = (c_d, r x c_d).  Per node, with S = sum over its links to p of 6 w_d rho_f c_d c_d^T
// and [r] the matrix of r x .: Z_VV = S, Z_OmegaV = [r] S, Z_OmegaOmega = [r] S [r]^T.  G is
// summed from the deviations f~_d - w_d rho_f (the rest part 2 rho_f sum w_d c_d and S come
// from counts of links per direction class), the sums over the chunk in FP64 in a fixed
// order; the motion kernel adds the chunks in chunk order and solves for (V, Omega).
// A stale chunk's entries are found again first (rebuild_chunk).  Each lane then takes the
// entries of its rank and reads the populations of the entry's link directions at the node's
// own slot: the entries are in (z, y, x) order, so along a row neighbouring lanes read
// neighbouring values.  Bound by those gathers and their latency.  (Records of G per node and
// slot, written by a kernel over every listed node and gathered here, cost 30 + 18 us on the
// FCC wave case (FP64 45 + 25) against 31 us (48) for this kernel, 23 us without stale slabs: the records
// took a pass over the link words of every node and 16 bytes per link node each way.)
// FUSED: one workgroup per particle, a wave per chunk and a ninth for p's contacts meanwhile
// and its motion (motion_update) after the workgroup's barrier.  This saves the motion kernel's
// launch and its loads, but a workgroup holds its place until the motion is done, so it pays
// while every workgroup has a CU of its own, which a set's room for particles bounds (FCC packings, FP32, us for links and motion, fused
// | apart: 256 particles 19 | 25, 384 28 | 28, 512 32 | 30, 768 41 | 34; 60 in a chain, FP64,
// 14 | 19).  Otherwise a workgroup per four slabs, first the equatorial slabs of every
// particle, which hold most of the entries, then the polar ones (in slab order the long waves
// of the last workgroups ran alone: 39 us instead of 36 on the FCC wave case), and the motion
// kernel after.  A set with more than kChunks chunks a particle is not fused.
constexpr int kFusedParticles = 256;
constexpr int links_waves(bool fused) { return fused ? kChunks : kChunks / 2; }
template <int P, bool NR, bool FUSED>
__global__ __launch_bounds__(64 * (links_waves(FUSED) + (FUSED ? 1 : 0))) __attribute__((amdgpu_waves_per_eu(NR ? 3 : 5)))
void k_links(DevSet s)
{
    using S = typename Prec<P>::S;
    using C = typename Prec<P>::C;
    constexpr int kWaves = links_waves(FUSED);
    __shared__ int l_cells[kWaves][kCellLds], l_c[kWaves][kLinkLds];
    __shared__ unsigned l_g[kWaves][kLinkLds];
    __shared__ int2 l_segs[kWaves][256];
    // FUSED: the sums of the chunks (F0, sum xr x G, then the link-set sums), added in chunk order
    __shared__ double l_sum[FUSED ? kChunks : 1][kLinkComp + kZComp], l_lp[kLinkComp + kZComp], l_work[kMotionWork];
    static_assert(kLinkComp + kZComp <= 64, "one lane per component");
    const long long t = *s.tstep;
    const int par = (int)(t & 1);
    const int lane = threadIdx.x & 63, wv = (int)(threadIdx.x >> 6);
    if (s.ptot == 0) return;
    // particles in XCD order, neighbours sharing lines of the populations (45 us in launch
    // order on the FCC wave case, then 32)
    // (not fused: row `part` of the grid takes the two slabs next on either side of the ones of
    // the rows before)
    const int chunks = FUSED ? kChunks : s.chunks;
    const int part = FUSED ? 0 : (int)blockIdx.y, mid = chunks / 2, side = kWaves / 2;
    const int p = uni(xcd_swizzle((int)blockIdx.x, s.ptot));
    const int chunk = uni(FUSED ? wv : (wv < side ? mid - side * (part + 1) + wv : mid + side * (part - 1) + wv));
    if (FUSED && wv == kWaves) {
        const MemberDev *M = s.mem + uni(s.pmem[p]);
        if (p - uni(M->p_off) >= uni(M->np)) return; // (every wave of the workgroup)
        const MotionRow row = motion_row(s, p, par);
        const double con = contact_pass(s, M, p, par, 0);
        __syncthreads();
        if (lane < kLinkComp + kZComp) {
            double v = 0.0;
#pragma unroll
            for (int q = 0; q < kChunks; ++q) v += l_sum[FUSED ? q : 0][lane];
            l_lp[lane] = v;
        }
        wave_fence();
        motion_update(s, M, p, par, t, row, con, l_lp, l_work);
        return;
    }
    // the chunk's state is loaded together with p's lattice, before the checks that need
    // the lattice (everything here is indexed by p < ptot)
    const int m = uni(s.pmem[p]);
    const double *Xo = s.X[par];
    const double X0 = Xo[3 * p], X1 = Xo[3 * p + 1], X2 = Xo[3 * p + 2];
    const double R0 = s.Xref[3 * p], R1 = s.Xref[3 * p + 1], R2 = s.Xref[3 * p + 2];
    // (a list rebuild under compact storage moves the nodes' storage slots)
    const bool stale = (s.lreb[p] == t - 1) || (s.ldirty[p * chunks + chunk] == t - 1) ||
                       (s.compact && *s.relist_at == t);
    int cntx = s.xcnt[p * chunks + chunk];
    const MemberDev *M = s.mem + m;
    const int pl = p - uni(M->p_off);
    if (pl >= uni(M->np)) return;
    double *sums = FUSED ? l_sum[chunk] : s.ppart + ((long long)p * chunks + chunk) * kLinkComp;
    if (stale)
        cntx = rebuild_chunk<NR>(s, M, p, chunk, chunks, X0, X1, X2, l_cells[wv], l_segs[wv], l_c[wv], l_g[wv],
                                 FUSED ? sums + kLinkComp : nullptr);
    else if (FUSED && lane < kZComp)
        sums[kLinkComp + lane] = s.zcache[((long long)p * chunks + chunk) * kZComp + lane];
    const bool in_lds = stale && cntx <= kLinkLds; // (the wave's own LDS)

    const int nx = uni(M->nx), ny = uni(M->ny);
    const int per0 = uni(M->per[0]), per1 = uni(M->per[1]), per2 = uni(M->per[2]);
    const double box0 = uni(M->box[0]), box1 = uni(M->box[1]), box2 = uni(M->box[2]);
    const unsigned nc = (unsigned)uni(M->ncell);
    const S *A = (const S *)(par ? s.popB : s.popA) + uni(M->pop_off);
    const double rho_f = uni(M->rho_f);
    const bool rest_free = uni(M->rest_free) != 0;
    const int nxy = nx * ny;
    const long long lbase = ((long long)p * chunks + chunk) * s.xcap;
    const int *xc = s.xcell + lbase;
    const int *xs = s.xslot + lbase;
    const unsigned *xg = s.xgrp + lbase;
    const double inv_nxy = 1.0 / (double)nxy, inv_nx = 1.0 / (double)nx;

    // Positions of the entries' nodes relative to the particle's reference point X_ref,
    // xr = x - X_ref (minimum image; X_ref moves only with the slabs, which rebuilds the
    // entries).  With delta = X - X_ref, r = xr - delta, so the torque is
    // sum xr x G - delta x F0, and Z follows from sums over the link set alone:
    // S = sum S_n, Qx = sum [xr] S_n, Wx = sum [xr] S_n [xr]^T (the motion kernel applies delta).
    const double a18 = 2.0 * rho_f / 18.0, a36 = 2.0 * rho_f / 36.0;   // 2 rho_f w_d
    // (in a set with a narrow lattice the entry's image of p is the one that holds its link
    // group: its arm from the current centre X, as group_arm, plus the small displacement
    // X - X_ref)
    const double dX0 = mimg(X0 - R0, per0, box0), dX1 = mimg(X1 - R1, per1, box1), dX2 = mimg(X2 - R2, per2, box2);
    auto rel_pos = [&](int cell, unsigned g, double &x0, double &x1, double &x2) {
        const int kk = div_uni(cell, nxy, inv_nxy), rem = cell - kk * nxy;
        const int jj = div_uni(rem, nx, inv_nx), ii = rem - jj * nx;
        if constexpr (NR) {
            group_arm<true>(M, g, ii, jj, kk, X0, X1, X2, x0, x1, x2);
            x0 += dX0; x1 += dX1; x2 += dX2;
        } else {
            x0 = mimg((double)ii - R0, per0, box0);
            x1 = mimg((double)jj - R1, per1, box1);
            x2 = mimg((double)kk - R2, per2, box2);
        }
    };

    // F0 = sum 2 c_d f~_d and sum xr x (the node's part of F0) over the entries
    double acc[kLinkComp];
#pragma unroll
    for (int c = 0; c < kLinkComp; ++c) acc[c] = 0.0;
    // (the entries of the next round are loaded while this round's populations are)
    struct Entry { int cell; unsigned at, g; };
    auto entry = [&](int k) {
        const int kv = k < cntx ? k : 0;
        Entry en;
        if (in_lds) {
            en.cell = l_c[wv][kv];
            en.at = (unsigned)max(l_cells[wv][kv], 0);
            en.g = k < cntx ? l_g[wv][kv] : 0u;
        } else {
            en.cell = xc[kv];
            en.at = (unsigned)max(xs[kv], 0); // (a node with links is fluid, hence listed)
            const unsigned g = xg[kv];
            en.g = k < cntx ? g : 0u;
        }
        return en;
    };
    Entry next = entry(lane);
    for (int base = 0; base < cntx; base += 64) {
        const int cell = next.cell;
        const unsigned at = next.at, g = next.g;
        // every lane loads for every direction, a lane without the link the array's first
        // element (one shared line)
        S raw[kQ - 1];
#pragma unroll
        for (int e = 0; e < kQ - 1; ++e) raw[e] = ldo(A, ((g >> e) & 1u) ? (unsigned)kOPP[e] * nc + at : 0u);
        next = entry(base + 64 + lane);
        if (g == 0u) continue;
        // G = sum c_d (f~_d - w_d rho_f), in the collision precision
        C D0 = C(0), D1 = C(0), D2 = C(0);
#pragma unroll
        for (int e = 0; e < kQ - 1; ++e) {
            const int d = kOPP[e];
            const C v = ((g >> e) & 1u) ? decode_dev<P>(raw[e], d, rho_f) : C(0);
            if (kCX[d] > 0) D0 += v; else if (kCX[d] < 0) D0 -= v;
            if (kCY[d] > 0) D1 += v; else if (kCY[d] < 0) D1 -= v;
            if (kCZ[d] > 0) D2 += v; else if (kCZ[d] < 0) D2 -= v;
        }
        // sum 2 c_d f~_d = 2 G + 2 rho_f sum w_d c_d
        auto rest = [&](int axis) {
            const int na = (int)__popc(g & link_mask(axis, 1, false)) - (int)__popc(g & link_mask(axis, -1, false));
            const int nd = (int)__popc(g & link_mask(axis, 1, true)) - (int)__popc(g & link_mask(axis, -1, true));
            return a18 * (double)na + a36 * (double)nd;
        };
        // (rest_free: without the rest state's part)
        const double G0 = 2.0 * (double)D0 + (rest_free ? 0.0 : rest(0));
        const double G1 = 2.0 * (double)D1 + (rest_free ? 0.0 : rest(1));
        const double G2 = 2.0 * (double)D2 + (rest_free ? 0.0 : rest(2));
        double x0, x1, x2;
        rel_pos(cell, g, x0, x1, x2);
        acc[0] += G0; acc[1] += G1; acc[2] += G2;
        acc[3] += x1 * G2 - x2 * G1;
        acc[4] += x2 * G0 - x0 * G2;
        acc[5] += x0 * G1 - x1 * G0;
    }
#pragma unroll
    for (int c = 0; c < kLinkComp; ++c) acc[c] = wave_sum(acc[c]);
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < kLinkComp; ++c) sums[c] = acc[c];
    }
    if constexpr (FUSED) __syncthreads();
}

// ---------------------------------------------------------------------------
// re-projection kernel
// ---------------------------------------------------------------------------
// Per-particle context of the re-projection: the particle, its lattice, its position
// after this step's motion (mode 0) or now (mode 1), and its near neighbours (staged in
// the workgroup's shared memory, slot w).
struct RemapCtx {
    int p, w, nn;
    const MemberDev *M;
    double X[3], R, R2;
    int per[3];
    double box[3];
};

constexpr int kRemapWaves = 4; // particles per workgroup of the re-projection kernel

// Particles beyond kRestRadius are watched while they move less than kRestStep a step (a shell
// of kRestShell on both sides of the surface holds 8 pi R^2 kRestShell nodes, 9 at R = 60).
constexpr double kRestStep = 5e-5, kRestShell = 1e-4;

// Re-projection (Sec. 2.3), one wave per particle.  The nodes whose owner the step can have
// changed lie within the particle's displacement of its surface, or inside it within the
// overlap depth with a neighbour; they are found row by row from the sphere's equation (a
// few FP32 operations per row and no memory, about 360 rows at R = 8.5), queued, and
// evaluated exactly 64 at a time.  Bound by the latency of its few dependent loads.  (Shell
// and surface-band lists per particle, read every step and built again by a whole workgroup
// once the particle had left its shell, cost 25 us per step on the FCC wave case and 370 us
// on a suspension of 288 moving spheres, where some list was always being built, against
// 16 and 26 us.)  Waves never synchronise; workgroups past the particles reduce the probe planes.
template <int P, bool WATCH>
__global__ __launch_bounds__(256) void k_remap(DevSet s, int mode, int only)
{
    using S = typename Prec<P>::S;
    __shared__ double red[4][8];
    __shared__ double nbw[kRemapWaves][kNearCap][4];
    __shared__ int nbidw[kRemapWaves][kNearCap];
    // each wave's queue of candidate nodes
    constexpr int kQueue = 256;
    __shared__ int qcell[kRemapWaves][kQueue];
    // the step being completed (mode 0), copied by the refresh kernel, or by the fluid kernel of a
    // set that runs no refresh; the counter itself is advanced here and read by no workgroup of
    // this kernel
    const long long t = (mode == 0) ? *s.tcopy : *s.tstep;
    const int par = (int)(t & 1);
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int npw = (s.ptot + kRemapWaves - 1) / kRemapWaves;
    if (mode == 0 && blockIdx.x == 0 && tid == 0) *s.tstep = t + 1;

    if ((int)blockIdx.x >= npw) {
        // probe plane reduction, one workgroup per (lattice, probe), tiles in fixed order
        if (mode != 0) return;
        const int q = blockIdx.x - npw;
        if (q >= s.nprobe_total) return;
        int m = 0;
        while (m + 1 < s.nmem && s.mem[m + 1].plist_off <= q) ++m;
        while (s.mem[m].n_probe == 0 || q - s.mem[m].plist_off >= s.mem[m].n_probe) ++m;
        const MemberDev *Mq = s.mem + m;
        const int k = q - Mq->plist_off;
        const int z = s.plist[Mq->plist_off + k];
        const int tz = z / s.nzt, dz = z - tz * s.nzt;
        const int ntile = Mq->ntx * Mq->nty;
        double v[4] = {0, 0, 0, 0};
        for (int c = tid; c < ntile; c += 256) {
            const long long gt = Mq->tile_off + (long long)tz * ntile + c;
            const double *pp = s.pprt + (gt * s.nzt + dz) * 4;
            v[0] += pp[0]; v[1] += pp[1]; v[2] += pp[2]; v[3] += pp[3];
        }
        block_sum<4>(v, red);
        if (tid == 0) {
            double *o = s.ring + Mq->ring_off + ((t % s.ring_len) * Mq->n_probe + k) * 4;
            o[0] = v[0]; o[1] = v[1]; o[2] = v[2]; o[3] = v[3];
        }
        return;
    }

    const int sp = (mode == 1) ? par : (par ^ 1); // buffers of the positions after the motion
    const double *Xs = s.X[sp], *Vs = s.V[sp], *Ws = s.W[sp];
    const int sn = par ^ 1;                       // population buffer holding f~(t+1)

    auto dist2c = [&](const RemapCtx &c, int i, int j, int k, double X0, double X1, double X2) {
        const double dx = mimg((double)i - X0, c.per[0], c.box[0]);
        const double dy = mimg((double)j - X1, c.per[1], c.box[1]);
        const double dz = mimg((double)k - X2, c.per[2], c.box[2]);
        return (dx * dx + dy * dy) + dz * dz;
    };

    // owner of one node after the motion; conversion of a covered node; opened: p uncovered it
    bool watch = false;         // a large particle that hardly moves, see below
    double gap = kRestShell;    // and the least distance of an evaluated node from its surface
    auto evaluate = [&](const RemapCtx &c, int ii, int jj, int kk, int cell, double (&acc)[6], int &conv,
                        bool &opened) {
        const MemberDev *M = c.M;
        const int p = c.p;
        const int *cur = s.own[par] + M->cell_off;
        const int was = cur[cell];
        const double d2n = dist2c(c, ii, jj, kk, c.X[0], c.X[1], c.X[2]);
        if (WATCH && watch) gap = fmin(gap, fabs(sqrt(d2n) - c.R));
        // owner: smallest d^2, then smallest index, among the spheres containing the node
        int best = -1;
        double bd = 0.0;
        if (d2n <= c.R2) { best = p; bd = d2n; }
        for (int k = 0; k < c.nn; ++k) {
            const double dq = dist2c(c, ii, jj, kk, nbw[c.w][k][0], nbw[c.w][k][1], nbw[c.w][k][2]);
            if (dq <= nbw[c.w][k][3] * nbw[c.w][k][3]) {
                const int q = nbidw[c.w][k];
                if (best < 0 || dq < bd || (dq == bd && q < best)) { best = q; bd = dq; }
            }
        }
        if (mode == 1) {
            if (best >= 0) { s.own[0][M->cell_off + cell] = best; s.own[1][M->cell_off + cell] = best; }
            return;
        }
        if (best == was) return;
        s.own[par ^ 1][M->cell_off + cell] = best;
        // (the cached link entries that this change makes stale are marked by the next
        // refresh, which sees which link words actually change)
        const int slot = atomicAdd(s.chgcnt + par, 1);
        if (slot < s.chg_cap) {
            s.chg[par][2 * slot] = (int)(M->cell_off + cell);
            s.chg[par][2 * slot + 1] = best;
        } else {
            atomicOr(s.flags, 0x4u);
        }
        const double r0 = mimg((double)ii - c.X[0], c.per[0], c.box[0]);
        const double r1 = mimg((double)jj - c.X[1], c.per[1], c.box[1]);
        const double r2 = mimg((double)kk - c.X[2], c.per[2], c.box[2]);
        S *Bn = (S *)(sn ? s.popB : s.popA) + M->pop_off;
        const int nc = (int)M->ncell;
        const double rho_ff = M->rho_f;
        if (was < 0 && best == p) {
            // Eq. (convertFS): a covered node hands its momentum to the particle
            const int sl = node_slot(s, M, cell, ii, jj, kk);
            if (sl < 0) { atomicOr(s.flags, 0x100u); return; }
            double f[kQ];
#pragma unroll
            for (int d = 0; d < kQ; ++d) f[d] = (double)ld<P>(Bn, d * nc + sl, d, rho_ff);
            double rho, j0, j1, j2;
            moments<double>(f, rho, j0, j1, j2);
            conv = 1;
            acc[0] += j0; acc[1] += j1; acc[2] += j2;
            acc[3] += r1 * j2 - r2 * j1;
            acc[4] += r2 * j0 - r0 * j2;
            acc[5] += r0 * j1 - r1 * j0;
        }
        opened = was == p && best < 0;
    };

    // Eq. (convertSF): node `cell` uncovered by p is refilled with f^eq(rho_bar, V_b) and takes
    // rho_bar V_b from the particle; rho_bar averages the neighbours that are fluid before and
    // after the re-projection.  32 lanes per node: lane e < 18 takes neighbour e, so the node
    // maps, slots and populations of all neighbours are loaded together (one lane taking them
    // in turn cost 18 rounds of loads); then lane d < 19 stores population d.  Under compact
    // storage a node outside the lists has its refill parked for the list rebuild at the start
    // of the next step.  `on` is the same in a node's lanes.
    auto refill = [&](const RemapCtx &c, int cell, bool on, double (&acc)[6]) {
        const MemberDev *M = c.M;
        const int p = c.p, h = lane & 31;
        const int nx = M->nx, ny = M->ny, nz = M->nz, nxy = nx * ny, nc = (int)M->ncell;
        const int *cur = s.own[par] + M->cell_off;
        S *Bn = (S *)(sn ? s.popB : s.popA) + M->pop_off;
        const double rho_ff = M->rho_f;
        const int kk = cell / nxy, rem = cell - kk * nxy, jj = rem / nx, ii = rem - jj * nx;
        int xx = ii + dir_x(h), yy = jj + dir_y(h), zz = kk + dir_z(h);
        bool use = on && h < kQ - 1 && (c.per[0] || (xx >= 0 && xx < nx)) && (c.per[1] || (yy >= 0 && yy < ny)) &&
                   (c.per[2] || (zz >= 0 && zz < nz));
        xx = wrapc(xx, nx); yy = wrapc(yy, ny); zz = wrapc(zz, nz);
        const int yc = use ? (zz * ny + yy) * nx + xx : cell;
        const int ow = cur[yc];
        const int sl = s.compact ? slot_of(s, M, ii, jj, kk) : cell;
        int ys = s.compact ? slot_of(s, M, use ? xx : ii, use ? yy : jj, use ? zz : kk) : yc;
        use = use && ow < 0;
        if (use) {
            bool inside = dist2c(c, xx, yy, zz, c.X[0], c.X[1], c.X[2]) <= c.R2;
            for (int k = 0; k < c.nn && !inside; ++k)
                inside = dist2c(c, xx, yy, zz, nbw[c.w][k][0], nbw[c.w][k][1], nbw[c.w][k][2]) <=
                         nbw[c.w][k][3] * nbw[c.w][k][3];
            use = !inside;
            if (use && ys < 0) { atomicOr(s.flags, 0x100u); use = false; }
        }
        ys = use ? ys : 0;
        double rr = 0.0;
        {
            S raw[kQ];
#pragma unroll
            for (int d = 0; d < kQ; ++d) raw[d] = Bn[d * nc + ys];
            if (use)
#pragma unroll
                for (int d = 0; d < kQ; ++d) rr += (double)decode_full<P>(raw[d], d, rho_ff);
        }
        for (int off = 16; off >= 1; off >>= 1) rr += __shfl_xor(rr, off, 64);
        const unsigned long long bal = __ballot(use);
        const int cnt = __popc((unsigned)(lane < 32 ? bal : bal >> 32));
        if (!on) return;
        const double r0 = mimg((double)ii - c.X[0], c.per[0], c.box[0]);
        const double r1 = mimg((double)jj - c.X[1], c.per[1], c.box[1]);
        const double r2 = mimg((double)kk - c.X[2], c.per[2], c.box[2]);
        const double rbar = cnt > 0 ? rr / cnt : rho_ff;
        const double *Vp = Vs + 3 * p, *Wp = Ws + 3 * p;
        const double vb0 = Vp[0] + (Wp[1] * r2 - Wp[2] * r1);
        const double vb1 = Vp[1] + (Wp[2] * r0 - Wp[0] * r2);
        const double vb2 = Vp[2] + (Wp[0] * r1 - Wp[1] * r0);
        if (sl >= 0) {
            const double uu = vb0 * vb0 + vb1 * vb1 + vb2 * vb2;
            if (h < kQ) {
                const double cu = (double)dir_x(h) * vb0 + (double)dir_y(h) * vb1 + (double)dir_z(h) * vb2;
                const double w = h == kQ - 1 ? kWd[kQ - 1] : (h < 6 ? kWd[0] : kWd[6]);
                const double f = w * rbar * (1.0 + 3.0 * cu + 4.5 * (cu * cu) - 1.5 * uu);
                encode_full<P>(Bn + h * nc + sl, (typename Prec<P>::C)f, w, rho_ff);
            }
        } else if (h == 0) {
            const int pi = atomicAdd(s.pcnt + par, 1);
            if (pi < kPendCap) {
                double *rec = s.pbuf[par] + 4 * pi;
                rec[0] = rbar; rec[1] = vb0; rec[2] = vb1; rec[3] = vb2;
                s.pend[M->cell_off + cell] = pi;
                *s.relist_at = t + 1;
                atomicOr(s.flags, 0x200u);
            } else {
                atomicOr(s.flags, 0x100u);
            }
        }
        if (h == 0) {
            const double m0 = rbar * vb0, m1 = rbar * vb1, m2 = rbar * vb2;
            acc[0] -= m0; acc[1] -= m1; acc[2] -= m2;
            acc[3] -= r1 * m2 - r2 * m1;
            acc[4] -= r2 * m0 - r0 * m2;
            acc[5] -= r0 * m1 - r1 * m0;
        }
    };

    const int p = blockIdx.x * kRemapWaves + wv;
    if (p >= s.ptot) return;
    // Per-particle values that depend on nothing else are loaded together: the member, the
    // near list, the reference states, and p's position in both buffers.
    const int m = s.pmem[p];
    const int nn = min(s.nnear[p], kNearCap);
    const int q_near = s.nearl[(long long)p * kNearCap + (lane & (kNearCap - 1))];
    const double R = s.R[p];
    const double Xr[3] = {s.Xref[3 * p], s.Xref[3 * p + 1], s.Xref[3 * p + 2]};
    const double Xb0[3] = {s.X[0][3 * p], s.X[0][3 * p + 1], s.X[0][3 * p + 2]};
    const double Xb1[3] = {s.X[1][3 * p], s.X[1][3 * p + 1], s.X[1][3 * p + 2]};
    const double Xl[3] = {s.Xl[3 * p], s.Xl[3 * p + 1], s.Xl[3 * p + 2]};
    const double Xn[3] = {s.Xn[3 * p], s.Xn[3 * p + 1], s.Xn[3 * p + 2]};
    const MemberDev *M = s.mem + m;
    if (p - M->p_off >= M->np || (only >= 0 && m != only)) return;
    // (no wave stores the due step of a lattice whose near lists are due in this step)
    const bool near_build = mode == 0 && s.near_due[m] == t;
    const double skin = s.skin[m];
    RemapCtx c;
    c.p = p; c.w = wv; c.M = M;
    double Xold[3]; // the position of the node map being replaced
    for (int a = 0; a < 3; ++a) {
        c.per[a] = M->per[a];
        c.box[a] = M->box[a];
        c.X[a] = sp ? Xb1[a] : Xb0[a];
        Xold[a] = (mode == 1) ? c.X[a] : (par ? Xb1[a] : Xb0[a]);
    }
    c.R = R; c.R2 = R * R;
    c.nn = nn;
    auto dist = [&](const double *A, const double *B) {
        double v = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double d = mimg(A[a] - B[a], c.per[a], c.box[a]);
            v += d * d;
        }
        return sqrt(v);
    };
    // near neighbours (one lane each): positions staged for the wave, and the largest overlap
    // with p before and after the motion
    double dmax = 0.0;
    if (lane < nn) {
        const int q = q_near;
        const double Y[3] = {Xs[3 * q], Xs[3 * q + 1], Xs[3 * q + 2]}, Rq = s.R[q];
        nbidw[wv][lane] = q;
        nbw[wv][lane][0] = Y[0]; nbw[wv][lane][1] = Y[1]; nbw[wv][lane][2] = Y[2];
        nbw[wv][lane][3] = Rq;
        dmax = fmax(0.0, R + Rq - dist(Y, c.X));
        if (mode == 0) {
            const double *Z = s.X[par] + 3 * q;
            const double Yo[3] = {Z[0], Z[1], Z[2]};
            dmax = fmax(dmax, R + Rq - dist(Yo, Xold));
        }
    }
    for (int off = 32; off >= 1; off >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, off, 64));
    const double step = dist(c.X, Xold);
    // node lists: rebuilt at the start of the next step once p may have moved the skin
    if (s.listmode && lane == 0) {
        if (mode == 1) {
            *s.relist_at = t;
            const double *Vp = Vs + 3 * p;
            s.pspd[p] = sqrt(Vp[0] * Vp[0] + Vp[1] * Vp[1] + Vp[2] * Vp[2]);
        } else {
            // a node uncovered by the next re-projection should have a slot in the current
            // lists, so they are rebuilt while the particle stays within the skin after one
            // more step of up to list_margin times this step's displacement (under compact
            // storage a node uncovered outside them is parked until the rebuild)
            s.pspd[p] = step;
            if (dist(c.X, Xl) + s.list_margin * step >= skin - 1e-9) *s.relist_at = t + 1;
        }
    }
    // Candidates, by d = |x - X| after the motion: a node enters or leaves p only if |d - R|
    // <= the displacement; the order between p and an overlapping sphere changes only at
    // nodes of p within the overlap depth, before the motion (R - d <= depth + displacement)
    // or after it.  (At set-up every node inside p.)
    // A large particle that hardly moves and overlaps no other is watched: its search takes in
    // the nodes up to kRestShell off its surface and finds how far it may move before the first
    // of them can change, and until it has there is nothing to search.  (64 rows cost a wave 0.33
    // us; one sphere at rest, us per launch, searched | watched: radius 13 10.6 | 7.7, 18 14.6 |
    // 8, 36 35 | 9, 60 83 | 11, 100 212 | 11.  Up to a radius of 12 the search is short: 1.5 us
    // at 10.)
    const bool large = WATCH && mode == 0 && R > kRestRadius;
    double *rest = WATCH ? s.rest + 4 * (size_t)p : nullptr; // (the position of the last search and that distance)
    watch = large && step < kRestStep;
    bool quiet = false;
    if (watch && dmax == 0.0) {
        const double Xs0[3] = {rest[0], rest[1], rest[2]};
        quiet = dist(c.X, Xs0) + 1e-9 < rest[3];
    }
    const double mrg = row_margin(R) + (watch ? kRestShell : 0.0);
    const double outer = R + step + mrg, inner = (mode == 1) ? -1.0 : R - (dmax + step) - mrg;
    const float outer2 = (float)(outer * outer), inner2 = inner > 0.0 ? (float)(inner * inner) : -1.0f;
    const int nx = M->nx, ny = M->ny, nz = M->nz;
    int x0, x1, y0, y1, z0, z1;
    near_range(c.X[0], outer, nx, c.per[0], x0, x1);
    near_range(c.X[1], outer, ny, c.per[1], y0, y1);
    near_range(c.X[2], outer, nz, c.per[2], z0, z1);
    const int ix = (int)floor(c.X[0]);
    const float fx = (float)(c.X[0] - (double)ix);
    const int nj = max(y1 - y0 + 1, 0), nrow = quiet ? 0 : nj * max(z1 - z0 + 1, 0);
    const double inv_nj = 1.0 / (double)max(nj, 1);
    const int dxy = nx * ny;
    const double inv_dxy = 1.0 / (double)dxy, inv_nx = 1.0 / (double)nx;
    const unsigned long long below = (1ull << lane) - 1ull;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    int conv = 0, qn = 0;
    RowSpan r = {0, -1, 0, -1};
    int base_cell = 0, row0 = 0;
    for (;;) {
        const bool first = r.a0 <= r.a1, has = first || r.b0 <= r.b1;
        const unsigned long long bal = __ballot(has);
        if (bal == 0ull && row0 < nrow) {
            // the spans of the next 64 rows
            if (row0 + lane < nrow) {
                const int kz = div_uni(row0 + lane, nj, inv_nj), ky = row0 + lane - kz * nj;
                int zz = z0 + kz, yy = y0 + ky;
                const double dy = (double)yy - c.X[1], dz = (double)zz - c.X[2];
                r = row_span((float)(dy * dy + dz * dz), fx, inner2, outer2);
                r.a0 = max(r.a0, x0 - ix); r.b0 = max(r.b0, x0 - ix);
                r.a1 = min(r.a1, x1 - ix); r.b1 = min(r.b1, x1 - ix);
                if (c.per[1]) yy = yy < 0 ? yy + ny : (yy >= ny ? yy - ny : yy);
                if (c.per[2]) zz = zz < 0 ? zz + nz : (zz >= nz ? zz - nz : zz);
                base_cell = zz * dxy + yy * nx;
            }
            row0 += 64;
            continue;
        }
        if (has) {
            int x = ix + (first ? r.a0++ : r.b0++);
            if (c.per[0]) x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
            qcell[wv][qn + __popcll(bal & below)] = base_cell + x;
        }
        qn += __popcll(bal);
        if (bal != 0ull && qn <= kQueue - 64) continue;
        if (qn == 0) break; // no row and no node left
        wave_fence();
        // uncovered nodes go to the front of the queue (behind the round being evaluated)
        int on = 0;
        for (int q0 = 0; q0 < qn; q0 += 64) {
            const int q = q0 + lane;
            const int cell = q < qn ? qcell[wv][q] : 0;
            bool opened = false;
            if (q < qn) {
                const int kk = div_uni(cell, dxy, inv_dxy), rem = cell - kk * dxy;
                const int jj = div_uni(rem, nx, inv_nx), ii = rem - jj * nx;
                evaluate(c, ii, jj, kk, cell, acc, conv, opened);
            }
            const unsigned long long ob = __ballot(opened);
            wave_fence();
            if (opened) qcell[wv][on + __popcll(ob & below)] = cell;
            on += __popcll(ob);
        }
        wave_fence();
        for (int q = 0; q < on; q += 2) {
            const int at = q + (lane >> 5);
            refill(c, qcell[wv][min(at, on - 1)], at < on, acc);
        }
        conv |= on;
        // (the queue is filled again once every lane has read its entries)
        wave_fence();
        qn = 0;
    }
    if (large && !quiet) {
        const double g = watch ? wave_min_d(gap) : 0.0;
        if (lane < 4) rest[lane] = lane == 0 ? c.X[0] : lane == 1 ? c.X[1] : lane == 2 ? c.X[2] : g;
    } else if (WATCH && mode == 1 && lane == 0) {
        rest[3] = 0.0;
    }
    // the wave's conversion momentum (summed only when a lane made a conversion)
    if (__ballot(conv) != 0ull) {
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[k] = wave_sum(acc[k]);
    }
    if (lane == 0) {
        if (mode == 0)
            for (int a = 0; a < 3; ++a) { s.Ph[3 * p + a] = acc[a]; s.Lh[3 * p + a] = acc[3 + a]; }
        // the slabs of p's link entries, laid out around X at set-up and once it has moved
        // away from their reference point (the next link pass then finds its entries again)
        if (mode == 1 || dist(c.X, Xr) > kAnchorMove) {
            const double reach = R + kSlabReach + (fmin(dmax, kSlabLens) + 1e-9);
            int lo = (int)floor(c.X[2] - reach) - 1, hi = (int)ceil(c.X[2] + reach) + 1;
            if (!c.per[2]) { lo = max(lo, 0); hi = min(hi, nz - 1); }
            const int ext = c.per[2] ? min(hi - lo + 1, nz) : max(hi - lo + 1, 0);
            s.lzr[2 * p] = lo;
            s.lzr[2 * p + 1] = (ext + s.chunks - 1) / s.chunks;
            s.lreb[p] = (mode == 1) ? t - 1 : t;
            for (int a = 0; a < 3; ++a) s.Xref[3 * p + a] = c.X[a];
        }
    }
    if (mode == 1) {
        if (lane == 0)
            for (int a = 0; a < 3; ++a) s.Xn[3 * p + a] = c.X[a];
    } else if (!near_build) {
        if (lane == 0 && dist(c.X, Xn) > kNearMove) s.near_due[m] = t + 1;
    } else {
        // the near list from the positions after this step's motion: every particle within
        // R_p + R_q + kNearMargin, in index order
        const int q0 = M->p_off, nq = M->np;
        int near_total = 0;
#pragma unroll 4
        for (int base = 0; base < nq; base += 64) {
            const int q = q0 + min(base + lane, nq - 1);
            const double Y[3] = {Xs[3 * q], Xs[3 * q + 1], Xs[3 * q + 2]};
            const bool isnear = base + lane < nq && q != p && dist(Y, c.X) <= R + s.R[q] + kNearMargin;
            const unsigned long long bal = __ballot(isnear);
            if (isnear) {
                const int slot = near_total + __popcll(bal & below);
                if (slot < kNearCap) s.nearl[(long long)p * kNearCap + slot] = q;
                else atomicOr(s.flags, 0x2u);
            }
            near_total += __popcll(bal);
        }
        if (lane == 0) s.nnear[p] = min(near_total, kNearCap);
        if (lane == 0)
            for (int a = 0; a < 3; ++a) s.Xn[3 * p + a] = c.X[a];
    }
}

// ---------------------------------------------------------------------------
// initial populations f = w_d rho_f in both buffers
// ---------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(256) void k_init_pops(DevSet s, long long total_cells)
{
    using S = typename Prec<P>::S;
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= total_cells) return;
    const MemberDev *M = member_of_cell(s, c);
    const int cell = (int)(c - M->cell_off);
    const int nc = (int)M->ncell;
    S *A = (S *)s.popA + M->pop_off, *B = (S *)s.popB + M->pop_off;
    const double rho_ff = M->rho_f;
    for (int d = 0; d < kQ; ++d) {
        const typename Prec<P>::C v = (typename Prec<P>::C)(kWd[d] * M->rho_f);
        st<P>(A, d * nc + cell, d, v, rho_ff);
        st<P>(B, d * nc + cell, d, v, rho_ff);
    }
}

// ---------------------------------------------------------------------------
// macroscopic fields of one lattice (node layout): rho = sum_d f_d, rho u = sum_d f_d c_d
// (Eq. rhoAndU) in FP64, directions in index order; 0 at solid nodes.  out: [4][ncell].
// Compact storage is read at the nodes' slots, a fluid node outside the lists from its parked
// refill, rounded as it will be stored (spreading the set to the node layout first, and the
// list rebuild that the next step then owed, took 330 us on a 66 x 44 x 132 packing in FP64).
// ---------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(256) void k_fields(DevSet s, int m, double *out)
{
    const long long t = *s.tstep;
    const int par = (int)(t & 1);
    const MemberDev *M = s.mem + m;
    const long long nc = M->ncell;
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    using S = typename Prec<P>::S;
    const S *A = (const S *)(par ? s.popB : s.popA) + M->pop_off;
    double rho = 0.0, j0 = 0.0, j1 = 0.0, j2 = 0.0;
    if (s.own[par][M->cell_off + c] < 0) {
        const double rho_ff = M->rho_f;
        const int nx = M->nx, nxy = nx * M->ny, z = (int)c / nxy, rem = (int)c - z * nxy;
        const int sl = node_slot(s, M, (int)c, rem % nx, rem / nx, z);
        S raw[kQ];
#pragma unroll
        for (int d = 0; d < kQ; ++d) raw[d] = A[(unsigned)(d * nc + max(sl, 0))];
        if (sl < 0) {
            const int pi = s.pend[M->cell_off + c];
            double rb = rho_ff, u0 = 0.0, u1 = 0.0, u2 = 0.0;
            if (pi >= 0) {
                const double *rec = s.pbuf[par ^ 1] + 4 * pi;
                rb = rec[0]; u0 = rec[1]; u1 = rec[2]; u2 = rec[3];
            }
            const double uu = u0 * u0 + u1 * u1 + u2 * u2;
#pragma unroll
            for (int d = 0; d < kQ; ++d)
                st<P>(raw, d, d, (typename Prec<P>::C)feq(d, rb, u0, u1, u2, uu), rho_ff);
        }
#pragma unroll
        for (int d = 0; d < kQ; ++d) {
            const double f = (double)ld<P>(raw, d, d, rho_ff);
            rho += f;
            j0 += f * kCXd[d];
            j1 += f * kCYd[d];
            j2 += f * kCZd[d];
        }
        j0 /= rho; j1 /= rho; j2 /= rho;
    }
    out[c] = rho;
    out[nc + c] = j0;
    out[2 * nc + c] = j1;
    out[3 * nc + c] = j2;
}

// X, V, Omega, F_h, T_h of particles [p0, p0 + n), 3 n values each: one copy to the host
// instead of a read of the step counter and five copies (one step of a sphere in a 32^3 box and
// its state back on the host, 172 -> 100 us)
__global__ __launch_bounds__(256) void k_particles_out(DevSet s, int p0, int n, double *out)
{
    const int par = (int)(*s.tstep & 1);
    const double *src[5] = {s.X[par], s.V[par], s.W[par], s.Fh, s.Th};
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= 3 * n) return;
#pragma unroll
    for (int q = 0; q < 5; ++q) out[(long long)q * 3 * n + k] = src[q][3ll * p0 + k];
}

// ---------------------------------------------------------------------------
// compact storage back to the node layout (before the host reads or writes populations,
// or replaces particles): per plane, listed nodes move from their slots to their nodes,
// every other node takes the rest state w_d rho_f, and the row tables become the identity
// ---------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(256) void k_expand(DevSet s)
{
    using S = typename Prec<P>::S;
    const long long t = *s.tstep;
    const int par = (int)(t & 1);
    for (int pl = blockIdx.x; pl < s.nplanes; pl += gridDim.x) {
        int lo = 0, hi = s.nmem - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s.mem[mid].pz_off <= pl) lo = mid;
            else hi = mid - 1;
        }
        const MemberDev *M = s.mem + lo;
        const int z = pl - M->pz_off, nx = M->nx, ny = M->ny, nxy = nx * ny, nw = M->nw;
        const long long nc = M->ncell;
        S *A = (S *)(par ? s.popB : s.popA) + M->pop_off;
        S *Cb = (S *)s.popC + M->pop_off;
        const double rho_ff = M->rho_f;
        const long long z0 = (long long)z * nxy;
        // the list of this plane is the one the row tables were built from
        for (int c = threadIdx.x; c < nxy; c += blockDim.x) {
            const int j = c / nx, i = c - j * nx;
            const int sl = slot_of(s, M, i, j, z);
            if (sl >= 0)
                for (int d = 0; d < kQ; ++d) Cb[d * nc + z0 + c] = A[d * nc + sl];
        }
        __threadfence_block();
        __syncthreads();
        for (int c = threadIdx.x; c < nxy; c += blockDim.x) {
            const int j = c / nx, i = c - j * nx;
            if (slot_of(s, M, i, j, z) >= 0) {
                for (int d = 0; d < kQ; ++d) A[d * nc + z0 + c] = Cb[d * nc + z0 + c];
            } else {
                // a parked refill of the last re-projection, else the rest state
                const long long gcell = M->cell_off + z0 + c;
                const int pi = s.pend[gcell];
                double rb = M->rho_f, u0 = 0.0, u1 = 0.0, u2 = 0.0;
                if (pi >= 0) {
                    const double *rec = s.pbuf[par ^ 1] + 4 * pi;
                    rb = rec[0]; u0 = rec[1]; u1 = rec[2]; u2 = rec[3];
                    s.pend[gcell] = -1;
                }
                const double uu = u0 * u0 + u1 * u1 + u2 * u2;
                for (int d = 0; d < kQ; ++d)
                    st<P>(A, (unsigned)(d * nc + z0 + c), d, (typename Prec<P>::C)feq(d, rb, u0, u1, u2, uu), rho_ff);
            }
        }
        __syncthreads();
        uint2 *rtp = s.rt + M->rt_off + (long long)z * ny * nw;
        for (int w = threadIdx.x; w < ny * nw; w += blockDim.x) {
            const int j = w / nw, x0 = (w - j * nw) * 32;
            const int nb = min(32, nx - x0);
            rtp[w] = make_uint2(nb == 32 ? 0xffffffffu : ((1u << nb) - 1u), (unsigned)(j * nx + x0));
        }
        // the plane's list no longer describes the layout: the next rebuild lays it out
        if (threadIdx.x == 0) s.ccnt[pl] = -1;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// adjoint of the fluid step over frozen particle geometry
// ---------------------------------------------------------------------------
// The window's forward map is the fluid step with the node map and the particles frozen
// (positions, angular velocities; prescribed velocities V): pull streaming with
// stationary walls and the moving walls of Eq. (mem), the density faces (Sec. 2.4) with
// rho_in = rho_f + A s(t+1), and the BGK collision, all on deviations from the rest
// state as in the coupled fluid kernel.  Its discrete adjoint propagates a loss gradient
// on the probe signals backwards: lambda^n = (dS/df^n)^T lambda^{n+1} + dL/df^n.

//
// The geometry is frozen, so the window works on its fluid nodes alone, numbered by slot
// with x fastest, with one occupancy word and the slot of the word's first node per 32 nodes
// of a row (the row table).  Along a row fluid nodes hold consecutive slots, so the
// 18 sources of a node come from nine row words.  A slot carries the directions that bounce
// back (mask.x) and those of them whose source lies in a particle (mask.y), the link
// directions; per link, packed in slot order from loff, the term of the moving wall (wall,
// filled once per forward) and the sum of dL/dg0 over the window (macc).
// Bound by HBM: a forward step reads and writes 19 populations a fluid node, an adjoint step
// reads 19 populations and 19 adjoint values and writes 19.  On the 64 x 64 x 256 packing of
// 275 spheres (459 000 fluid nodes, FP64) a forward step takes 29 us (28 at the rate of a
// device copy) and an adjoint step 65 us (48, of which 6 for the link sums); FP32 18 and
// 52 us.  One thread per cell of the lattice with an owner lookup per direction, probe sums
// by one workgroup per plane and mu and lambda in two kernels took 187 + 493 and 837 + 105
// us.  (Holding the adjoint step to 168 VGPRs for a third wave per SIMD spills: 127 us.)

__device__ __forceinline__ int adj_unknown(const AdjDev &a, int k)
{
    // the directions a density face leaves unknown: c_z = +1 at the lower face, -1 at the upper
    int m = 0;
#pragma unroll
    for (int e = 0; e < kQ - 1; ++e) {
        if (kCZ[e] > 0 && k == 0 && a.M.bc[4] == BC_PRESSURE) m |= 1 << e;
        if (kCZ[e] < 0 && k == a.M.nz - 1 && a.M.bc[5] == BC_PRESSURE) m |= 1 << e;
    }
    return m;
}

__device__ __forceinline__ void adj_coords(const AdjDev &a, int cell, int &i, int &j, int &k)
{
    const int nxy = a.M.nx * a.M.ny;
    k = cell / nxy;
    const int rem = cell - k * nxy;
    j = rem / a.M.nx;
    i = rem - j * a.M.nx;
}

// The source of direction e of cell (i, j, k): its cell index, or -1 for a wall, -2 for a
// source outside a density face.
__device__ __forceinline__ int adj_source_cell(const AdjDev &a, int e, int i, int j, int k)
{
    const MemberDev &M = a.M;
    const int dims[3] = {M.nx, M.ny, M.nz};
    int c[3] = {i - kCXd[e], j - kCYd[e], k - kCZd[e]};
    int kind = 0;
    for (int ax = 0; ax < 3; ++ax) {
        if (c[ax] < 0 || c[ax] >= dims[ax]) {
            const int f = M.bc[2 * ax + (c[ax] >= dims[ax] ? 1 : 0)];
            if (f == BC_PRESSURE) kind = 2;
            else if (f == BC_WALL) kind = max(kind, 1);
            else c[ax] = c[ax] < 0 ? c[ax] + dims[ax] : c[ax] - dims[ax];
        }
    }
    if (kind != 0) return -kind;
    return (c[2] * dims[1] + c[1]) * dims[0] + c[0];
}

// Sum of v over the threads before this one in the workgroup (256 threads) and the total.
__device__ __forceinline__ int block_scan(int v, int &total, int *cnt4)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int inc = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(inc, off, 64);
        if (lane >= off) inc += o;
    }
    if (lane == 63) cnt4[wv] = inc;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wv; ++w) before += cnt4[w];
    total = cnt4[0] + cnt4[1] + cnt4[2] + cnt4[3];
    __syncthreads();
    return before + inc - v;
}

// Window set-up (1): frozen node map with local particle indices, occupancy words, and the
// number of fluid nodes of each plane; one workgroup per plane.
__global__ __launch_bounds__(256) void k_adj_rows(AdjDev a, const int *own)
{
    __shared__ int cnt4[4];
    const int z = blockIdx.x, nx = a.M.nx, ny = a.M.ny, nxy = nx * ny, nw = a.M.nw;
    for (int c = threadIdx.x; c < nxy; c += 256) {
        const int o = own[z * nxy + c];
        a.own[z * nxy + c] = o < 0 ? -1 : o - a.M.p_off;
    }
    int count = 0;
    for (int w = threadIdx.x; w < ny * nw; w += 256) {
        const int j = w / nw, x0 = (w - j * nw) * 32;
        unsigned bits = 0u;
        for (int b = 0; b < min(32, nx - x0); ++b)
            if (own[z * nxy + j * nx + x0 + b] < 0) bits |= 1u << b;
        a.rows[z * ny * nw + w] = make_uint2(bits, 0u);
        count += __popc(bits);
    }
    int total;
    (void)block_scan(count, total, cnt4);
    if (threadIdx.x == 0) a.pbase[z] = total;
}

// (2) first slot of each plane; pbase[nz] the number of fluid nodes, nlink cleared.
__global__ __launch_bounds__(256) void k_adj_planes(AdjDev a)
{
    __shared__ int cnt4[4];
    int run = 0;
    for (int z0 = 0; z0 < a.M.nz; z0 += 256) {
        const int z = z0 + (int)threadIdx.x;
        int total;
        const int before = block_scan(z < a.M.nz ? a.pbase[z] : 0, total, cnt4);
        if (z < a.M.nz) a.pbase[z] = run + before;
        run += total;
    }
    if (threadIdx.x == 0) {
        a.pbase[a.M.nz] = run;
        *a.nlink = 0;
    }
}

// (3) slots of the row words and the node of each slot; one workgroup per plane.
__global__ __launch_bounds__(256) void k_adj_slots(AdjDev a)
{
    __shared__ int cnt4[4];
    const int z = blockIdx.x, nx = a.M.nx, ny = a.M.ny, nxy = nx * ny, nw = a.M.nw;
    int run = a.pbase[z];
    for (int w0 = 0; w0 < ny * nw; w0 += 256) {
        const int w = w0 + (int)threadIdx.x;
        const unsigned bits = w < ny * nw ? a.rows[z * ny * nw + w].x : 0u;
        int total;
        int at = run + block_scan(__popc(bits), total, cnt4);
        if (w < ny * nw) {
            a.rows[z * ny * nw + w].y = (unsigned)at;
            const int j = w / nw, x0 = (w - j * nw) * 32;
            for (unsigned m = bits; m; m &= m - 1u) a.node[at++] = z * nxy + j * nx + x0 + __ffs(m) - 1;
        }
        run += total;
    }
}

// (4) bounce-back and link directions of each slot, and where its links are packed (the
// waves take their ranges in any order: only sums of a link's own values depend on it).
__global__ __launch_bounds__(256) void k_adj_masks(AdjDev a)
{
    const int r = blockIdx.x * 256 + (int)threadIdx.x, lane = threadIdx.x & 63;
    unsigned back = 0u, link = 0u;
    if (r < a.nf) {
        int i, j, k;
        adj_coords(a, a.node[r], i, j, k);
        for (int e = 0; e < kQ - 1; ++e) {
            const int sc = adj_source_cell(a, e, i, j, k);
            if (sc == -1) back |= 1u << e;
            else if (sc >= 0 && a.own[sc] >= 0) { back |= 1u << e; link |= 1u << e; }
        }
    }
    const int n = __popc(link);
    int inc = n;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(inc, off, 64);
        if (lane >= off) inc += o;
    }
    int base = 0;
    if (lane == 63) base = atomicAdd(a.nlink, inc);
    base = __shfl(base, 63, 64);
    if (r >= a.nf) return;
    a.mask[r] = make_uint2(back, link);
    a.loff[r] = base + inc - n;
}

// (5) the start populations (node layout, stride ncell) at their slots.
template <typename T>
__global__ __launch_bounds__(256) void k_adj_start(AdjDev a, const T *src, T *dst)
{
    const int r = blockIdx.x * 256 + (int)threadIdx.x;
    if (r >= a.nf) return;
    const int cell = a.node[r];
    for (int d = 0; d < kQ; ++d) dst[(size_t)d * a.ns + r] = src[(size_t)d * a.ncell + cell];
}

// Per forward: the moving-wall term of Eq. (mem) of every link, 2 (w_d / c_s^2) rho_f V_b . c_d
// with V_b . c_d = c_d . (V + Omega x (x - X)) of the source's particle.
template <int P>
__global__ __launch_bounds__(256) void k_adj_wall(AdjDev a)
{
    using C = typename Prec<P>::C;
    const int r = blockIdx.x * 256 + (int)threadIdx.x;
    if (r >= a.nf) return;
    const unsigned link = a.mask[r].y;
    if (link == 0u) return;
    const MemberDev &M = a.M;
    int i, j, k;
    adj_coords(a, a.node[r], i, j, k);
    C *w = static_cast<C *>(a.wall) + a.loff[r];
    for (unsigned m = link; m; m &= m - 1u) {
        const int e = __ffs(m) - 1;
        const int q = a.own[adj_source_cell(a, e, i, j, k)];
        // (on a narrow lattice, from the link's midpoint, which fixes the image, as group_arm)
        const double h0 = M.narrow ? 0.5 * kCXd[e] : 0.0, h1 = M.narrow ? 0.5 * kCYd[e] : 0.0,
                     h2 = M.narrow ? 0.5 * kCZd[e] : 0.0;
        const double r0 = mimg(((double)i - h0) - a.X[3 * q], M.per[0], M.box[0]) + h0;
        const double r1 = mimg(((double)j - h1) - a.X[3 * q + 1], M.per[1], M.box[1]) + h1;
        const double r2 = mimg(((double)k - h2) - a.X[3 * q + 2], M.per[2], M.box[2]) + h2;
        const double *V = a.V + 3 * q, *W = a.W + 3 * q;
        const double u0 = V[0] + (W[1] * r2 - W[2] * r1);
        const double u1 = V[1] + (W[2] * r0 - W[0] * r2);
        const double u2 = V[2] + (W[0] * r1 - W[1] * r0);
        // c_d = -c_e
        const double cu = -(double)kCXd[e] * u0 - (double)kCYd[e] * u1 - (double)kCZd[e] * u2;
        *w++ = (C)((e < 6 ? kMW[0] : kMW[6]) * a.rho_f) * (C)cu;
    }
}

// Element of the population arrays each direction of slot r is pulled from: f~_e at the
// source, or f~_{e*} at r itself from a wall or a particle (for an unknown direction of a
// density face: its own element, whose value is not used).
__device__ __forceinline__ void adj_sources(const AdjDev &a, int i, int j, int k, unsigned r, unsigned back, unsigned unk,
                                            unsigned (&idx)[kQ - 1])
{
    const int nx = a.M.nx, ny = a.M.ny, nz = a.M.nz, nw = a.M.nw, per_x = a.M.per[0];
    const unsigned ns = (unsigned)a.ns, b = 1u << (i & 31);
    const int wx = (i == 0) ? nx - 1 : 0; // the x neighbour across a periodic face
    const unsigned bw = 1u << (wx & 31);
    uint2 wv[9], ww[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int row = (wrapc(k + q % 3 - 1, nz) * ny + wrapc(j + q / 3 - 1, ny)) * nw;
        wv[q] = a.rows[row + (i >> 5)];
        ww[q] = per_x ? a.rows[row + (wx >> 5)] : make_uint2(0u, 0u);
    }
#pragma unroll
    for (int e = 0; e < kQ - 1; ++e) {
        const int q = (1 - kCY[e]) * 3 + (1 - kCZ[e]);
        const unsigned rk = wv[q].y + (unsigned)__popc(wv[q].x & (b - 1u));
        unsigned v;
        if (kCX[e] == 0) {
            v = rk;
        } else {
            const unsigned rwr = ww[q].y + (unsigned)__popc(ww[q].x & (bw - 1u));
            if (kCX[e] < 0) v = (i < nx - 1) ? rk + ((wv[q].x & b) ? 1u : 0u) : rwr;
            else v = (i > 0) ? rk - 1u : rwr;
        }
        const unsigned far = (unsigned)e * ns + v;
        idx[e] = ((back >> e) & 1u) ? (unsigned)kOPP[e] * ns + r : (((unk >> e) & 1u) ? (unsigned)e * ns + r : far);
    }
}

// Element idx of a window's [19][ns] array.  FP64 and FP32 arrays stay below 4 GiB (as the
// set's), so a 32-bit byte offset from a scalar base reaches them.  A 16-bit set's FP32
// adjoint fields can be larger.
template <int P, typename T>
__device__ __forceinline__ T adj_ld(const T *base, unsigned idx)
{
    if constexpr (P == PREC_FP64 || P == PREC_FP32) return ldo(base, idx);
    else return base[idx];
}
template <int P, typename T>
__device__ __forceinline__ void adj_st(T *base, unsigned idx, T v)
{
    if constexpr (P == PREC_FP64 || P == PREC_FP32) sto(base, idx, v);
    else base[idx] = v;
}

// Pre-collision populations (deviations from the rest state) of slot r, density faces
// included, pulled from the state fin.  ALL: the moving-wall terms are loaded for every
// direction at once instead of behind a branch per direction; the adjoint step, whose waves
// are few (212 VGPRs), gains by it (72.6 -> 65.3 us), the forward step does not (29.3 -> 30.8).
template <int P, bool ALL>
__device__ __forceinline__ void adj_gather(const AdjDev &a, const typename Prec<P>::S *fin, int k, unsigned r,
                                           const unsigned (&idx)[kQ - 1], unsigned link, unsigned unk, int n,
                                           typename Prec<P>::C (&g)[kQ])
{
    using C = typename Prec<P>::C;
    using S = typename Prec<P>::S;
    S raw[kQ];
#pragma unroll
    for (int e = 0; e < kQ - 1; ++e) raw[e] = adj_ld<P>(fin, idx[e]);
    raw[kQ - 1] = adj_ld<P>(fin, (unsigned)(kQ - 1) * (unsigned)a.ns + r);
#pragma unroll
    for (int e = 0; e < kQ; ++e) g[e] = ((unk >> e) & 1u) ? C(0) : decode_dev<P>(raw[e], e, a.rho_f);
    if (link) {
        const C *w = static_cast<const C *>(a.wall) + a.loff[r];
        if constexpr (ALL) {
            // (a lane without a link at e reads the next link's term, or past the last one
            // within the array's capacity)
            C t[kQ - 1];
#pragma unroll
            for (int e = 0; e < kQ - 1; ++e) t[e] = w[__popc(link & ((1u << e) - 1u))];
#pragma unroll
            for (int e = 0; e < kQ - 1; ++e) g[e] -= ((link >> e) & 1u) ? t[e] : C(0);
        } else {
#pragma unroll
            for (int e = 0; e < kQ - 1; ++e)
                if ((link >> e) & 1u) g[e] -= w[__popc(link & ((1u << e) - 1u))];
        }
    }
    if (k == 0 && a.M.bc[4] == BC_PRESSURE) zou_he<C>(g, (C)(a.amp * a.shape[n]), false);
    if (k == a.M.nz - 1 && a.M.bc[5] == BC_PRESSURE) zou_he<C>(g, C(0), true);
}

// One frozen forward step fin -> fout (no store after the window's last step, whose end
// state nothing reads), and per wave of a probe plane its sum of rho - rho_f before the
// collision, at row m of the partial sums.
template <int P>
__global__ __launch_bounds__(256) void k_adj_step(AdjDev a, const typename Prec<P>::S *fin, typename Prec<P>::S *fout,
                                                  int n, int m)
{
    using C = typename Prec<P>::C;
    const int blk = xcd_swizzle((int)blockIdx.x, (int)gridDim.x);
    const unsigned r = (unsigned)blk * 256 + threadIdx.x;
    const bool on = (int)r < a.nf;
    int i = 0, j = 0, k = 0;
    if (on) adj_coords(a, a.node[r], i, j, k);
    const int pidx = on ? a.pzm[k] : -1;
    if (!fout && __ballot(pidx >= 0) == 0ull) return;
    const uint2 mk = on ? a.mask[r] : make_uint2(0x3ffffu, 0u);
    const unsigned unk = (unsigned)adj_unknown(a, k);
    unsigned idx[kQ - 1];
    adj_sources(a, i, j, k, on ? r : 0u, mk.x, unk, idx);
    C f[kQ];
    adj_gather<P, false>(a, fin, k, on ? r : 0u, idx, mk.y, unk, n, f);
    C drho, jx, jy, jz;
    moments<C>(f, drho, jx, jy, jz);
    // the wave's sum for each probe plane it holds nodes of
    for (unsigned long long left = __ballot(pidx >= 0); left != 0ull;) {
        const int lead = __ffsll((long long)left) - 1, kk = __shfl(k, lead, 64), pp = __shfl(pidx, lead, 64);
        const bool mine = pidx == pp;
        const double sum = wave_sum(mine ? (double)drho : 0.0);
        if ((int)(threadIdx.x & 63) == lead)
            a.part[((size_t)m * a.n_probe + pp) * a.wpp + ((int)(r >> 6) - (a.pbase[kk] >> 6))] = sum;
        left &= ~__ballot(mine);
    }
    if (!fout || !on) return;
    const C rho = (C)a.rho_f + drho;
    const C ux = jx / rho, uy = jy / rho, uz = jz / rho;
    const C uu = ux * ux + uy * uy + uz * uz;
    const C om = (C)a.omega;
#pragma unroll
    for (int d = 0; d < kQ; ++d) {
        const C fe = feq_dev<C>(d, drho, rho, ux, uy, uz, uu);
        store_dev<P>(fout + (size_t)d * a.ns, r, d, f[d] + om * (fe - f[d]), a.rho_f);
    }
}

// Probe signals of steps n0 + m, m from m0 on: the waves' sums of each plane in order, over
// the plane's fluid nodes; one wave per (plane, step).
__global__ __launch_bounds__(64) void k_adj_signal(AdjDev a, int n0, int m0)
{
    const int kp = blockIdx.x, m = m0 + (int)blockIdx.y, k = a.probe_z[kp];
    const int s0 = a.pbase[k], s1 = a.pbase[k + 1], nwv = s1 > s0 ? ((s1 - 1) >> 6) - (s0 >> 6) + 1 : 0;
    const double *p = a.part + ((size_t)m * a.n_probe + kp) * a.wpp;
    double v = 0.0;
    for (int w = threadIdx.x; w < nwv; w += 64) v += p[w];
    v = wave_sum(v);
    if (threadIdx.x == 0) a.P[(long long)(n0 + m) * a.n_probe + kp] = v / a.probe_nfl[kp];
}

// Fluid nodes of each probe plane (one workgroup per plane).
__global__ __launch_bounds__(256) void k_adj_nfl(AdjDev a, double *nfl)
{
    __shared__ double red[4][8];
    const int kp = blockIdx.x;
    if (kp >= a.n_probe) return;
    const int nxy = a.M.nx * a.M.ny;
    double v[1] = {0.0};
    for (int t = threadIdx.x; t < nxy; t += blockDim.x)
        if (a.own[a.probe_z[kp] * nxy + t] < 0) v[0] += 1.0;
    block_sum<1>(v, red);
    if (threadIdx.x == 0) nfl[kp] = v[0];
}

// Adjoint through step n at every fluid node: from lambda^{n+1} (dL/d of the post-collision
// state) and the probe term, mu = dL/dg0 of the pre-face populations g0 of time level
// n+1, written straight to lambda^n: every post-collision population has one consumer, the
// node that pulls it, so mu_e goes to the element direction e was pulled from (elements
// that leave through a density face have none and stay zero from the start of the backward
// pass).  Collision transpose: with A = sum lambda_d w_d, B = sum lambda_d w_d c_d,
// Cm = sum lambda_d w_d (c_d.u) c_d, D = sum lambda_d w_d (c_d.u)^2 (lattice units,
// 1/c_s^2 = 3), sum_d lambda_d df^eq_d/dg_e = A (1 + 1.5 u.u) - 4.5 D + (3 B + 9 Cm - 3 A u).c_e.
// The density faces are transposed by hand from their closure formulas.  Also collected:
// dL/domega = sum lambda_d (f^eq_d - g_d), dL/drho_in, and dL/dg0_e of every link (for dL/dV).
template <int P>
__global__ __launch_bounds__(256) void k_adj_back(AdjDev a, const typename Prec<P>::S *fin,
                                                  const typename Prec<P>::C *lam, typename Prec<P>::C *out, int n)
{
    using C = typename Prec<P>::C;
    __shared__ double red[4][8];
    const int blk = xcd_swizzle((int)blockIdx.x, (int)gridDim.x);
    const unsigned r = (unsigned)blk * 256 + threadIdx.x;
    const int ns = a.ns;
    double acc[2] = {0.0, 0.0}; // dL/domega, dL/drho_in
    if ((int)r < a.nf) {
        int i, j, k;
        adj_coords(a, a.node[r], i, j, k);
        const int pidx = a.pzm[k];
        const uint2 mk = a.mask[r];
        const unsigned unk = (unsigned)adj_unknown(a, k);
        unsigned idx[kQ - 1];
        adj_sources(a, i, j, k, r, mk.x, unk, idx);
        C l[kQ];
#pragma unroll
        for (int d = 0; d < kQ; ++d) l[d] = adj_ld<P>(lam, (unsigned)(d * ns) + r);
        C g[kQ];
        adj_gather<P, true>(a, fin, k, r, idx, mk.y, unk, n, g);
        const int face = (k == 0 && a.M.bc[4] == BC_PRESSURE) ? 0 : ((k == a.M.nz - 1 && a.M.bc[5] == BC_PRESSURE) ? 1 : -1);
        C drho, jx, jy, jz;
        moments<C>(g, drho, jx, jy, jz);
        const C rho = (C)a.rho_f + drho;
        const C ux = jx / rho, uy = jy / rho, uz = jz / rho;
        const C uu = ux * ux + uy * uy + uz * uz;
        C A = C(0), B0 = C(0), B1 = C(0), B2 = C(0), C0 = C(0), C1 = C(0), C2 = C(0), D = C(0);
        double gw = 0.0;
#pragma unroll
        for (int d = 0; d < kQ; ++d) {
            const C wl = (C)kWd[d] * l[d];
            const C cu = cdot(d, ux, uy, uz);
            const C wc = wl * cu;
            A += wl;
            if (kCX[d] > 0) { B0 += wl; C0 += wc; } else if (kCX[d] < 0) { B0 -= wl; C0 -= wc; }
            if (kCY[d] > 0) { B1 += wl; C1 += wc; } else if (kCY[d] < 0) { B1 -= wl; C1 -= wc; }
            if (kCZ[d] > 0) { B2 += wl; C2 += wc; } else if (kCZ[d] < 0) { B2 -= wl; C2 -= wc; }
            D += wc * cu;
            gw += (double)l[d] * (double)(feq_dev<C>(d, drho, rho, ux, uy, uz, uu) - g[d]);
        }
        acc[0] = gw;
        const C om = (C)a.omega;
        const C base = A * (C(1) + C(1.5) * uu) - C(4.5) * D;
        const C v0 = C(3) * B0 + C(9) * C0 - C(3) * A * ux;
        const C v1 = C(3) * B1 + C(9) * C1 - C(3) * A * uy;
        const C v2 = C(3) * B2 + C(9) * C2 - C(3) * A * uz;
        const C pt = pidx >= 0 ? (C)(a.dLdP[(long long)n * a.n_probe + pidx] / a.probe_nfl[pidx]) : C(0);
        C m[kQ];
#pragma unroll
        for (int e = 0; e < kQ; ++e) m[e] = (C(1) - om) * l[e] + om * (base + cdot(e, v0, v1, v2)) + pt;
        // density faces (paper index p -> m[p-1]); unknowns end with no dependence on g0
        if (face == 0) {
            const C av = m[4], bv = m[8], cv = m[12], dv = m[14], ev = m[16];
            const C R = av / C(3) + (bv + cv + dv + ev) / C(6), X = cv - bv, Y = ev - dv;
            acc[1] = (double)R * a.shape[n]; // d rho_in / dA = s(t+1)
            m[4] = m[8] = m[12] = m[14] = m[16] = C(0);
            const int s0[9] = {0, 1, 2, 3, 6, 7, 10, 11, 18}, sm[5] = {5, 9, 13, 15, 17};
#pragma unroll
            for (int q = 0; q < 9; ++q) m[s0[q]] -= R;
#pragma unroll
            for (int q = 0; q < 5; ++q) m[sm[q]] -= C(2) * R;
            m[0] += C(0.5) * X; m[6] += C(0.5) * X; m[7] += C(0.5) * X;
            m[1] -= C(0.5) * X; m[10] -= C(0.5) * X; m[11] -= C(0.5) * X;
            m[2] += C(0.5) * Y; m[6] += C(0.5) * Y; m[10] += C(0.5) * Y;
            m[3] -= C(0.5) * Y; m[7] -= C(0.5) * Y; m[11] -= C(0.5) * Y;
            m[5] += av; m[13] += bv; m[9] += cv; m[17] += dv; m[15] += ev;
        } else if (face == 1) {
            const C av = m[5], bv = m[13], cv = m[9], dv = m[17], ev = m[15];
            const C R = -av / C(3) - (bv + cv + dv + ev) / C(6), X = bv - cv, Y = dv - ev;
            m[5] = m[13] = m[9] = m[17] = m[15] = C(0);
            const int s0[9] = {0, 1, 2, 3, 6, 7, 10, 11, 18}, sp[5] = {4, 8, 12, 14, 16};
#pragma unroll
            for (int q = 0; q < 9; ++q) m[s0[q]] += R;
#pragma unroll
            for (int q = 0; q < 5; ++q) m[sp[q]] += C(2) * R;
            m[0] += C(0.5) * X; m[6] += C(0.5) * X; m[7] += C(0.5) * X;
            m[1] -= C(0.5) * X; m[10] -= C(0.5) * X; m[11] -= C(0.5) * X;
            m[2] += C(0.5) * Y; m[6] += C(0.5) * Y; m[10] += C(0.5) * Y;
            m[3] -= C(0.5) * Y; m[7] -= C(0.5) * Y; m[11] -= C(0.5) * Y;
            m[4] += av; m[8] += bv; m[12] += cv; m[14] += dv; m[16] += ev;
        }
        if (mk.y) {
            double *q = a.macc + a.loff[r], t[kQ - 1];
#pragma unroll
            for (int e = 0; e < kQ - 1; ++e) t[e] = q[__popc(mk.y & ((1u << e) - 1u))];
#pragma unroll
            for (int e = 0; e < kQ - 1; ++e)
                if ((mk.y >> e) & 1u) q[__popc(mk.y & ((1u << e) - 1u))] = t[e] + (double)m[e];
        }
#pragma unroll
        for (int e = 0; e < kQ - 1; ++e)
            if (!((unk >> e) & 1u)) adj_st<P>(out, idx[e], m[e]);
        adj_st<P>(out, (unsigned)((kQ - 1) * ns) + r, m[kQ - 1]);
    }
    block_sum<2>(acc, red);
    if (threadIdx.x == 0) {
        a.acc_w[blk] += acc[0];
        a.acc_a[blk] += acc[1];
    }
}

// dL/dV_q = sum over q's links (x, e) of -2 (w_d / c_s^2) rho_f c_d dL/dg0_e(x), d = e*:
// one workgroup per particle over the nodes within R_q + 2 of X_q, in a fixed order (16
// waves: with few particles the kernel is a chain of loads per node, 4 waves took 359 us
// for 275 spheres of radius 8).
constexpr int kVgradThreads = 1024;
__global__ __launch_bounds__(kVgradThreads) void k_adj_vgrad(AdjDev a)
{
    __shared__ double red[kVgradThreads / 64][3];
    const int q = blockIdx.x;
    if (q >= a.np) return;
    const MemberDev &M = a.M;
    const int dims[3] = {M.nx, M.ny, M.nz};
    int lo[3], ext[3];
    for (int ax = 0; ax < 3; ++ax) axis_range(a.X[3 * q + ax], a.R[q] + 2.0, dims[ax], M.per[ax], lo[ax], ext[ax]);
    const int tot = ext[0] * ext[1] * ext[2];
    double acc[3] = {0.0, 0.0, 0.0};
    for (int idx = threadIdx.x; idx < tot; idx += kVgradThreads) {
        const int ii = wrapc(lo[0] + idx % ext[0], dims[0]);
        const int jj = wrapc(lo[1] + (idx / ext[0]) % ext[1], dims[1]);
        const int kk = wrapc(lo[2] + idx / (ext[0] * ext[1]), dims[2]);
        const uint2 w = a.rows[(kk * dims[1] + jj) * M.nw + (ii >> 5)];
        const unsigned b = 1u << (ii & 31);
        if (!(w.x & b)) continue; // solid
        const unsigned r = w.y + (unsigned)__popc(w.x & (b - 1u));
        const unsigned link = a.mask[r].y;
        const double *mr = a.macc + a.loff[r];
        for (unsigned m = link; m; m &= m - 1u, ++mr) {
            const int e = __ffs(m) - 1;
            if (a.own[adj_source_cell(a, e, ii, jj, kk)] != q) continue;
            // d g0_e / dV = -2 (w_d / c_s^2) rho_f c_d with c_d = -c_e and w_d = w_e
            const double wd = (e < 6) ? 1.0 / 18.0 : 1.0 / 36.0;
            const double f = 2.0 * wd / kCS2 * a.rho_f * *mr;
            acc[0] += f * kCXd[e];
            acc[1] += f * kCYd[e];
            acc[2] += f * kCZd[e];
        }
    }
    for (int ax = 0; ax < 3; ++ax) {
        const double v = wave_sum(acc[ax]);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][ax] = v;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double v = 0.0;
        for (int w = 0; w < kVgradThreads / 64; ++w) v += red[w][threadIdx.x];
        a.gv[3 * q + threadIdx.x] = v;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <bool CMP, bool NR>
void *fluid_ptr(int prec)
{
    switch (prec) {
    case PREC_FP64: return (void *)&k_fluid<PREC_FP64, CMP, NR>;
    case PREC_FP32: return (void *)&k_fluid<PREC_FP32, CMP, NR>;
    case PREC_FP16DEV: return (void *)&k_fluid<PREC_FP16DEV, CMP, NR>;
    default: return (void *)&k_fluid<PREC_BF16DEV, CMP, NR>;
    }
}
void *fluid_kernel_ptr(int prec, int compact, int narrow)
{
    if (narrow) return compact ? fluid_ptr<true, true>(prec) : fluid_ptr<false, true>(prec);
    return compact ? fluid_ptr<true, false>(prec) : fluid_ptr<false, false>(prec);
}
template <bool NR, bool FUSED>
void *links_ptr(int prec)
{
    switch (prec) {
    case PREC_FP64: return (void *)&k_links<PREC_FP64, NR, FUSED>;
    case PREC_FP32: return (void *)&k_links<PREC_FP32, NR, FUSED>;
    case PREC_FP16DEV: return (void *)&k_links<PREC_FP16DEV, NR, FUSED>;
    default: return (void *)&k_links<PREC_BF16DEV, NR, FUSED>;
    }
}
bool links_fused(const DevSet &s) { return s.ptot <= kFusedParticles && s.chunks == kChunks; }
void *links_kernel_ptr(int prec, const DevSet &s)
{
    if (s.narrow) return links_fused(s) ? links_ptr<true, true>(prec) : links_ptr<true, false>(prec);
    return links_fused(s) ? links_ptr<false, true>(prec) : links_ptr<false, false>(prec);
}
void *motion_kernel_ptr(const DevSet &s) { return s.chunks > kChunks ? (void *)&k_motion<true> : (void *)&k_motion<false>; }
template <bool WATCH>
void *remap_ptr(int prec)
{
    switch (prec) {
    case PREC_FP64: return (void *)&k_remap<PREC_FP64, WATCH>;
    case PREC_FP32: return (void *)&k_remap<PREC_FP32, WATCH>;
    case PREC_FP16DEV: return (void *)&k_remap<PREC_FP16DEV, WATCH>;
    default: return (void *)&k_remap<PREC_BF16DEV, WATCH>;
    }
}
void *remap_kernel_ptr(int prec, const DevSet &s) { return s.rest ? remap_ptr<true>(prec) : remap_ptr<false>(prec); }
dim3 links_grid(const DevSet &s) { return dim3(max(s.ptot, 1), links_fused(s) ? 1 : s.chunks / links_waves(false)); }
int refresh_grid(const DevSet &) { return kRefreshBlocks; }
void *refresh_kernel_ptr(int prec)
{
    switch (prec) {
    case PREC_FP64: return reinterpret_cast<void *>(&k_refresh<PREC_FP64>);
    case PREC_FP32: return reinterpret_cast<void *>(&k_refresh<PREC_FP32>);
    case PREC_FP16DEV: return reinterpret_cast<void *>(&k_refresh<PREC_FP16DEV>);
    default: return reinterpret_cast<void *>(&k_refresh<PREC_BF16DEV>);
    }
}

hipError_t launch_refresh(int prec, const DevSet &s, hipStream_t st)
{
    const dim3 g(refresh_grid(s)), b(256);
    switch (prec) {
    case PREC_FP64: hipLaunchKernelGGL(k_refresh<PREC_FP64>, g, b, 0, st, s); break;
    case PREC_FP32: hipLaunchKernelGGL(k_refresh<PREC_FP32>, g, b, 0, st, s); break;
    case PREC_FP16DEV: hipLaunchKernelGGL(k_refresh<PREC_FP16DEV>, g, b, 0, st, s); break;
    default: hipLaunchKernelGGL(k_refresh<PREC_BF16DEV>, g, b, 0, st, s); break;
    }
    return hipGetLastError();
}
int motion_grid(const DevSet &s) { return max((s.ptot + kMotionWaves - 1) / kMotionWaves, 1); }
int remap_grid(const DevSet &s) { return max((s.ptot + kRemapWaves - 1) / kRemapWaves + s.nprobe_total, 1); }

hipError_t launch_fluid(int prec, const DevSet &s, hipStream_t st)
{
    hipLaunchKernelGGL(reinterpret_cast<void (*)(DevSet)>(fluid_kernel_ptr(prec, s.compact, s.narrow)),
                       dim3(s.tiles_total), dim3(256), 0, st, s);
    return hipGetLastError();
}

int links_block(const DevSet &s) { return links_fused(s) ? 64 * (links_waves(true) + 1) : 64 * links_waves(false); }

hipError_t launch_links(int prec, const DevSet &s, hipStream_t st)
{
    hipLaunchKernelGGL(reinterpret_cast<void (*)(DevSet)>(links_kernel_ptr(prec, s)), links_grid(s),
                       dim3(links_block(s)), 0, st, s);
    return hipGetLastError();
}

hipError_t launch_motion(const DevSet &s, int mode, int only_member, hipStream_t st)
{
    hipLaunchKernelGGL(reinterpret_cast<void (*)(DevSet, int, int)>(motion_kernel_ptr(s)), dim3(motion_grid(s)),
                       dim3(64 * kMotionWaves), 0, st, s, mode, only_member);
    return hipGetLastError();
}

hipError_t launch_remap(int prec, const DevSet &s, int mode, int only_member, hipStream_t st)
{
    hipLaunchKernelGGL(reinterpret_cast<void (*)(DevSet, int, int)>(remap_kernel_ptr(prec, s)), dim3(remap_grid(s)),
                       dim3(256), 0, st, s, mode, only_member);
    return hipGetLastError();
}

int adj_blocks(const AdjDev &a) { return (a.ns + 255) / 256; }

template <int P> using StoreT = typename Prec<P>::S;
template <int P> using CompT = typename Prec<P>::C;

hipError_t launch_adj_geometry(const AdjDev &a, const int *own, hipStream_t st)
{
    hipLaunchKernelGGL(k_adj_rows, dim3(a.M.nz), dim3(256), 0, st, a, own);
    hipLaunchKernelGGL(k_adj_planes, dim3(1), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_adj_slots, dim3(a.M.nz), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_adj_start(int prec, const AdjDev &a, const void *src, void *dst, hipStream_t st)
{
    if (a.n_probe > 0) hipLaunchKernelGGL(k_adj_nfl, dim3(a.n_probe), dim3(256), 0, st, a, (double *)a.probe_nfl);
    if (a.ns == 0) return hipGetLastError();
    const dim3 g(adj_blocks(a)), b(256);
    hipLaunchKernelGGL(k_adj_masks, g, b, 0, st, a);
    switch (prec) {
    case PREC_FP64: hipLaunchKernelGGL(k_adj_start<double>, g, b, 0, st, a, (const double *)src, (double *)dst); break;
    case PREC_FP32: hipLaunchKernelGGL(k_adj_start<float>, g, b, 0, st, a, (const float *)src, (float *)dst); break;
    default: hipLaunchKernelGGL(k_adj_start<uint16_t>, g, b, 0, st, a, (const uint16_t *)src, (uint16_t *)dst); break;
    }
    return hipGetLastError();
}

template <int P> hipError_t adj_wall_p(const AdjDev &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_adj_wall<P>, dim3(adj_blocks(a)), dim3(256), 0, st, a);
    return hipGetLastError();
}
template <int P> hipError_t adj_step_p(const AdjDev &a, const void *fin, void *fout, int n, int m, hipStream_t st)
{
    hipLaunchKernelGGL(k_adj_step<P>, dim3(adj_blocks(a)), dim3(256), 0, st, a, (const StoreT<P> *)fin, (StoreT<P> *)fout,
                       n, m);
    return hipGetLastError();
}
template <int P>
hipError_t adj_back_p(const AdjDev &a, const void *fin, const void *lam, void *out, int n, hipStream_t st)
{
    hipLaunchKernelGGL(k_adj_back<P>, dim3(adj_blocks(a)), dim3(256), 0, st, a, (const StoreT<P> *)fin,
                       (const CompT<P> *)lam, (CompT<P> *)out, n);
    return hipGetLastError();
}

hipError_t launch_adj_wall(int prec, const AdjDev &a, hipStream_t st)
{
    if (a.ns == 0) return hipSuccess;
    switch (prec) {
    case PREC_FP64: return adj_wall_p<PREC_FP64>(a, st);
    case PREC_FP32: return adj_wall_p<PREC_FP32>(a, st);
    case PREC_FP16DEV: return adj_wall_p<PREC_FP16DEV>(a, st);
    default: return adj_wall_p<PREC_BF16DEV>(a, st);
    }
}

hipError_t launch_adj_step(int prec, const AdjDev &a, const void *fin, void *fout, int n, int m, hipStream_t st)
{
    if (a.ns == 0) return hipSuccess;
    switch (prec) {
    case PREC_FP64: return adj_step_p<PREC_FP64>(a, fin, fout, n, m, st);
    case PREC_FP32: return adj_step_p<PREC_FP32>(a, fin, fout, n, m, st);
    case PREC_FP16DEV: return adj_step_p<PREC_FP16DEV>(a, fin, fout, n, m, st);
    default: return adj_step_p<PREC_BF16DEV>(a, fin, fout, n, m, st);
    }
}

hipError_t launch_adj_signal(const AdjDev &a, int n0, int count, hipStream_t st)
{
    if (a.n_probe == 0 || count == 0) return hipSuccess;
    // (one grid row per step of the segment: rows of a grid are few, so in parts)
    for (int m = 0; m < count; m += 32768)
        hipLaunchKernelGGL(k_adj_signal, dim3(a.n_probe, min(32768, count - m)), dim3(64), 0, st, a, n0, m);
    return hipGetLastError();
}

hipError_t launch_adj_back(int prec, const AdjDev &a, const void *fin, const void *lam, void *out, int n, hipStream_t st)
{
    if (a.ns == 0) return hipSuccess;
    switch (prec) {
    case PREC_FP64: return adj_back_p<PREC_FP64>(a, fin, lam, out, n, st);
    case PREC_FP32: return adj_back_p<PREC_FP32>(a, fin, lam, out, n, st);
    case PREC_FP16DEV: return adj_back_p<PREC_FP16DEV>(a, fin, lam, out, n, st);
    default: return adj_back_p<PREC_BF16DEV>(a, fin, lam, out, n, st);
    }
}

hipError_t launch_adj_vgrad(const AdjDev &a, hipStream_t st)
{
    if (a.np > 0) hipLaunchKernelGGL(k_adj_vgrad, dim3(a.np), dim3(kVgradThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_particles_out(const DevSet &s, int p0, int n, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_particles_out, dim3((3 * n + 255) / 256), dim3(256), 0, st, s, p0, n, out);
    return hipGetLastError();
}

hipError_t launch_init_pops(int prec, const DevSet &s, long long total_cells, hipStream_t st)
{
    const unsigned grid = (unsigned)((total_cells + 255) / 256);
    if (grid == 0) return hipSuccess;
    switch (prec) {
    case PREC_FP64: hipLaunchKernelGGL(k_init_pops<PREC_FP64>, dim3(grid), dim3(256), 0, st, s, total_cells); break;
    case PREC_FP32: hipLaunchKernelGGL(k_init_pops<PREC_FP32>, dim3(grid), dim3(256), 0, st, s, total_cells); break;
    case PREC_FP16DEV: hipLaunchKernelGGL(k_init_pops<PREC_FP16DEV>, dim3(grid), dim3(256), 0, st, s, total_cells); break;
    default: hipLaunchKernelGGL(k_init_pops<PREC_BF16DEV>, dim3(grid), dim3(256), 0, st, s, total_cells); break;
    }
    return hipGetLastError();
}

hipError_t launch_fields(int prec, const DevSet &s, int m, long long ncell, double *out, hipStream_t st)
{
    const dim3 g((unsigned)((ncell + 255) / 256)), b(256);
    switch (prec) {
    case PREC_FP64: hipLaunchKernelGGL(k_fields<PREC_FP64>, g, b, 0, st, s, m, out); break;
    case PREC_FP32: hipLaunchKernelGGL(k_fields<PREC_FP32>, g, b, 0, st, s, m, out); break;
    case PREC_FP16DEV: hipLaunchKernelGGL(k_fields<PREC_FP16DEV>, g, b, 0, st, s, m, out); break;
    default: hipLaunchKernelGGL(k_fields<PREC_BF16DEV>, g, b, 0, st, s, m, out); break;
    }
    return hipGetLastError();
}

hipError_t launch_expand(int prec, const DevSet &s, hipStream_t st)
{
    const dim3 g(max(s.nplanes, 1));
    switch (prec) {
    case PREC_FP64: hipLaunchKernelGGL(k_expand<PREC_FP64>, g, dim3(256), 0, st, s); break;
    case PREC_FP32: hipLaunchKernelGGL(k_expand<PREC_FP32>, g, dim3(256), 0, st, s); break;
    case PREC_FP16DEV: hipLaunchKernelGGL(k_expand<PREC_FP16DEV>, g, dim3(256), 0, st, s); break;
    default: hipLaunchKernelGGL(k_expand<PREC_BF16DEV>, g, dim3(256), 0, st, s); break;
    }
    return hipGetLastError();
}

} // namespace lbdem
