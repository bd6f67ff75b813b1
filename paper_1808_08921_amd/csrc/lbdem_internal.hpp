// lbdem_internal.hpp -- device-side data layout shared by the kernels and the host API.
//
// All device buffers of a set are carved out of one workspace.  Fields are SoA with x
// fastest.  Populations are double-buffered (A/B) and the node map, the particle state
// and the node-change list are double-buffered by the parity of the step counter that
// lives in device memory, so that a fixed sequence of kernel launches (a HIP graph)
// advances the set without host involvement.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbdem {

constexpr int kQ = 19;
constexpr int kNearCap = 32;       // near-neighbour table per particle
constexpr int kHistCap = 16;       // tangential contact history per particle
constexpr double kNearMargin = 3.0; // near list: |X_p - X_q| <= R_p + R_q + margin
// near lists are built again once a particle of the lattice has moved this far since they
// were: two particles then close by less than 2 (0.15 + 0.25 + 0.25) = 1.3 before the new
// lists take effect, and a sphere that contains a neighbour node of a particle's swept node
// lies within R_p + R_q + 0.25 + sqrt(2) of it, together within the margin
constexpr double kNearMove = 0.15;
// a particle's slabs and the reference point of its link sums follow it after this distance
constexpr double kAnchorMove = 0.3;
// half height of a particle's slabs beyond its radius (plus the overlap depth up to
// kSlabLens, and one plane): a node with links lies within R + sqrt(2), and the particle
// within kAnchorMove, of the reference point.  The link sums are added slab by slab, so
// their rounding depends on this layout.
constexpr double kSlabReach = 2.0;
constexpr double kSlabLens = 1.0;
// node lists keep the solid nodes within a skin of a surface; the skin of a rebuild is
// kSkinSteps times the largest particle step of the lattice, within [kSkinMin, kListSkin]
constexpr double kListSkin = 0.25;
constexpr double kSkinMin = 0.05;
constexpr double kSkinSteps = 12.0;
constexpr int kPendCap = 16384;     // refills of unlisted nodes awaiting the next list rebuild
// z-slabs of the nodes around a particle, one wave of the link pass each; in sets of few large
// particles up to kMaxChunks (DevSet::chunks), so that a slab keeps to about kSlabPlanes planes
constexpr int kChunks = 8;
constexpr int kMaxChunks = 64;
constexpr int kSlabPlanes = 5;
// the re-projection watches particles beyond this radius that hardly move
constexpr double kRestRadius = 12.0;
// components of a link-pass partial per (particle, chunk): F0 (3) and sum xr x G (3), xr the
// node position relative to the particle's reference point
constexpr int kLinkComp = 6;
// cached link-set sums per (particle, chunk): S (6, upper triangle), Qx (9, row-major), Wx (6)
constexpr int kZComp = 21;
// Link words of a fluid node x (two 64-bit words per node: lw[c] and lw[ncell_total + c]).
// Word 0: bits 0-17 the directions e whose source x - c_e is inside a particle, bits 18-35
// the low bit of the slot (0..3) of the particle owning that source, bits 36-48 and 49-61
// the local indices of the particles in slots 0 and 1, bit 62 set when slots 2 or 3 are
// used, bit 63 when more than four particles border x.  Word 1: bits 0-17 the high slot
// bit per direction, bits 18-30 and 31-43 the local indices in slots 2 and 3.
constexpr int kMaxLocal = 8191;     // particles per lattice (13-bit local indices)
// workgroups of the start-of-step refresh kernel: as many as are resident at once at its 123
// registers (512 | 1024 | 2048: 17.0 | 11.6 | 11.7 us a step for 16 FCC lattices, 3.36 | 2.26 |
// 2.25 ms for their first lists; 135 | 115 | 114 us per rebuild of a settling suspension)
constexpr int kRefreshBlocks = 1024;
constexpr int kMaxPlaneWords = 8192; // row-table words of one x-y plane held in LDS (compact storage)
constexpr int kRtLds = 1536;        // row-table words a fluid-kernel workgroup stages in LDS (compact storage)

// Per-lattice constants (one entry per lattice of the set).
struct MemberDev {
    int nx, ny, nz;
    int bx_log2, bx, by;      // tile extent in x (power of two) and y; bx*by = 256
    int ntx, nty, ntz;        // tiles per axis
    int tile_off;             // first global tile index of this lattice
    int bc[6];                // face kinds
    int per[3];               // periodic axes
    double box[3];            // axis lengths as doubles
    long long ncell;          // nx*ny*nz
    long long cell_off;       // offset of this lattice in node-map arrays
    long long pop_off;        // offset of this lattice in population arrays (19*cell_off)
    double omega;             // 1/tau
    double rho_f;
    long long wave_off;       // offset in the waveform table (t_n + 2 entries)
    long long t_n;
    int pz_off;               // offset in the z -> probe-index map (nz entries)
    int plist_off;            // offset in the probe-plane list (n_probe entries)
    int n_probe;
    long long ring_off;       // offset (doubles) of this lattice's probe ring
    int p_off, p_cap, np;     // particles: global offset, capacity, current count
    double E, nu, mu, rho_p;
    int nw;                   // 32-node words per x row (compact storage)
    long long rt_off;         // offset of this lattice's row tables (compact storage)
    long long pv_from;        // first step whose particle velocities the ring holds for this lattice
    // 1: a periodic axis shorter than 2 max_radius + 4, where a fluid node can have links
    // into two images of one particle; its links are then grouped per (particle, image)
    // and the arm of a group is taken from the midpoint of one of its links
    int narrow;
    int rest_free;            // 1: link forces without the rest state's part (lbdem_params.rest_free)
};

// Everything a kernel needs, passed by value.
struct DevSet {
    int nmem;
    int fluid_off;            // 1: hydrodynamics switched off (particles feel contacts and F_g only)
    int narrow;               // 1: some lattice of the set is narrow (MemberDev::narrow)
    const MemberDev *mem;
    int tiles_total;
    int nzt;                  // z planes per fluid-kernel thread
    // node lists: per lattice and z plane, the listed nodes in x-fastest order at
    // [cell_off + z*nx*ny, +count); the fluid kernel then runs one thread per listed node
    int listmode;
    // compact storage (with node lists): populations of the listed nodes of plane z at
    // slots z*nx*ny + rank (rank in list order); row tables give, per x row and 32-node
    // word, the listed-node bits and the rank of the word's first listed node
    int compact;
    int es;                   // bytes per stored population value
    uint2 *rt;                // [sum over lattices of nz*ny*nw]
    void *popC;               // scratch population buffer for re-layouts
    int nplanes;              // sum of nz over the lattices
    int *clist;               // [ncell_total]
    int *ccnt;                // [sum of nz], indexed like the z -> probe map
    double *Xl;               // particle positions when the lists were built [ptot*3]
    long long *relist_at;     // step whose refresh rebuilds the lists
    double *skin;             // skin of each lattice's current lists [nmem]
    double list_margin;       // look-ahead of the rebuild trigger, in particle steps
    double *pspd;             // each particle's displacement in its last step [ptot]
    // compact storage: a node uncovered outside the lists has its refill (rho_bar, V_b)
    // parked until the next step's list rebuild: record index per node (-1 none)
    // [ncell_total], records [2][kPendCap*4] and counts [2] by the parity of the step
    int *pend;
    double *pbuf[2];
    int *pcnt;
    // populations
    void *popA, *popB;
    // node maps (index = parity), change lists (pairs cell, owner) and counts
    int *own[2];
    unsigned long long *lw;   // link words, two per node (all lattices) [2*ncell_total]
    // compact storage: the first link word of each listed node at its storage slot, or
    // kSolidWord for a listed solid node (the fluid kernel reads these in slot
    // order), and the step at which a full copy of the node map made them all stale
    unsigned long long *lwc;  // [ncell_total]
    long long *lwc_bad;
    long long ncell_total;
    // 64 bytes per node: the first half holds nothing between calls (the reads of particles and
    // fields gather into it, one at a time); the second half, in a set that may hold particles
    // beyond kRestRadius and where it has room for them, per particle the position of its last
    // full search by the re-projection and how far it may move from there before a node can
    // change (0: not known) [ptot*4], else null
    void *scratch;
    double *rest;
    int *chg[2];
    int chg_cap;
    int *chgcnt;              // [2]
    // probes
    double *pprt;             // [tiles_total*nzt*4]
    double *ring;
    int ring_len;
    const short *pzmap;
    const int *plist;
    int nprobe_total;
    const double *wave;
    // particles
    int ptot;
    double *X[2], *V[2], *W[2];
    double *R, *m, *I, *Fg, *Fh, *Th, *Ph, *Lh, *Xref;
    float *pf[2];             // FP32 wall state of the fluid kernel per particle (12 floats): X(t) and the
                              // velocities V, Omega of step t, at the parity of t
    int *fixed, *pmem;
    double *pvring;           // particle velocities after each step [pv_ring][ptot][3] (0 steps: none)
    int pv_ring;
    double *ppart;            // link-pass partials per (particle, chunk) [ptot*chunks*kLinkComp]
    double *zcache;           // link-set sums per (particle, chunk), rebuilt with its entries [ptot*chunks*kZComp]
    int *nearl, *nnear;       // [ptot*kNearCap], [ptot]
    long long *near_due;      // step whose re-projection builds a lattice's near lists [nmem]
    double *Xn;               // particle positions when its near list was built [ptot*3]
    // link entries: the nodes with links of a particle, per chunk in list order (z, y, x), at
    // [(p*chunks + chunk)*xcap, + xcnt[p*chunks + chunk])
    int chunks;               // chunks per particle, kChunks .. kMaxChunks (a multiple of kChunks)
    int xcap;
    int *xcell, *xcnt;
    int *xslot;               // storage slot of each cached entry's node
    unsigned *xgrp;           // the particle's link directions at each cached entry's node
    long long *lreb;          // step after which the particle's slabs were last laid out [ptot]
    long long *ldirty;        // last step in which link words of a chunk's nodes changed [ptot*chunks]
    // chunks are z-slabs around X_ref: first z (unwrapped) and slab height [ptot*2]
    int *lzr;
    int *hj[2];               // tangential history partner ids [ptot*kHistCap]
    double *hf[2];            // tangential history forces [ptot*kHistCap*3]
    int *hn[2];               // history counts [ptot]
    // counters
    long long *tstep;         // steps completed
    long long *tcopy;         // step in progress, for the re-projection kernel
    unsigned int *flags;
};

// Adjoint window over frozen geometry (one lattice): device view.  Populations and adjoint
// fields are [19][ns] over the window's slots (its fluid nodes, x fastest).
struct AdjDev {
    MemberDev M;              // the lattice's constants (offsets relative to this lattice)
    int ncell;
    int nf, ns;               // fluid nodes, and that rounded up to whole waves
    int *own;                 // frozen node map, local particle indices [ncell]
    uint2 *rows;              // per 32 nodes of a row: fluid bits, slot of the first fluid node [nz*ny*nw]
    int *pbase;               // first slot of each plane, then the number of fluid nodes [nz + 1]
    int *node;                // cell of each slot [nf]
    uint2 *mask;              // per slot: bounce-back directions, link directions [nf]
    int *loff;                // per slot: where its links are packed
    int *nlink;               // links packed so far
    void *wall;               // per link: moving-wall term of Eq. (mem) [nlink], collision precision
    const double *X, *W, *R;  // particle positions, angular velocities [np*3], radii [np]
    const double *V;          // particle velocities of the window [np*3]
    int np;
    double rho_f, omega, amp; // omega = 1/tau and the waveform amplitude of the window
    const double *shape;      // unit-amplitude waveform at time level t0+n+1 [nsteps]
    int n_probe;
    const int *probe_z;       // [n_probe]
    const short *pzm;         // probe index of each plane, -1 for none [nz]
    const double *probe_nfl;  // fluid nodes per probe plane [n_probe]
    int wpp;                  // most waves that hold nodes of one plane
    double *part;             // waves' density sums of the probe planes [ckpt_every][n_probe][wpp]
    double *P;                // probe signals [nsteps][n_probe]
    const double *dLdP;       // loss gradient [nsteps][n_probe]
    double *acc_w, *acc_a;    // per-workgroup sums of dL/domega and dL/dA [nblk]
    double *macc;             // summed dL/dg of every link [nlink]
    double *gv;               // dL/dV [np*3]
};

enum { BC_PERIODIC = 0, BC_WALL = 1, BC_PRESSURE = 2 };
enum { PREC_FP64 = 0, PREC_FP32 = 1, PREC_FP16DEV = 2, PREC_BF16DEV = 3 };

// kernel launchers (lbdem_kernels.hip)
hipError_t launch_refresh(int prec, const DevSet &s, hipStream_t st);
hipError_t launch_links(int prec, const DevSet &s, hipStream_t st);
hipError_t launch_motion(const DevSet &s, int mode, int only_member, hipStream_t st);
hipError_t launch_fluid(int prec, const DevSet &s, hipStream_t st);
hipError_t launch_remap(int prec, const DevSet &s, int mode, int only_member, hipStream_t st);
hipError_t launch_init_pops(int prec, const DevSet &s, long long total_cells, hipStream_t st);
hipError_t launch_expand(int prec, const DevSet &s, hipStream_t st);
hipError_t launch_particles_out(const DevSet &s, int p0, int n, double *out, hipStream_t st);
hipError_t launch_fields(int prec, const DevSet &s, int m, long long ncell, double *out, hipStream_t st);
// kernel entry points and grid sizes, for building HIP graphs
void *refresh_kernel_ptr(int prec);
bool links_fused(const DevSet &s); // the link kernel moves the particles too
void *links_kernel_ptr(int prec, const DevSet &s);
void *motion_kernel_ptr(const DevSet &s);
void *fluid_kernel_ptr(int prec, int compact, int narrow);
void *remap_kernel_ptr(int prec, const DevSet &s);
int refresh_grid(const DevSet &s);
dim3 links_grid(const DevSet &s);
int links_block(const DevSet &s);
int motion_grid(const DevSet &s);
int remap_grid(const DevSet &s);
// adjoint window kernels (lbdem_kernels.hip)
hipError_t launch_adj_geometry(const AdjDev &a, const int *own, hipStream_t st);
hipError_t launch_adj_start(int prec, const AdjDev &a, const void *src, void *dst, hipStream_t st);
hipError_t launch_adj_wall(int prec, const AdjDev &a, hipStream_t st);
hipError_t launch_adj_step(int prec, const AdjDev &a, const void *fin, void *fout, int n, int m, hipStream_t st);
hipError_t launch_adj_signal(const AdjDev &a, int n0, int count, hipStream_t st);
hipError_t launch_adj_back(int prec, const AdjDev &a, const void *fin, const void *lam, void *out, int n, hipStream_t st);
hipError_t launch_adj_vgrad(const AdjDev &a, hipStream_t st);
int adj_blocks(const AdjDev &a);


// dispersion analysis (lbdem_analysis.hip)
struct DftPlan {
    int nwb, ztiles, nzb, nchunk;     // frequency blocks, column tiles per block, column blocks, time chunks
    long long seg;                    // steps per wave of the time stage (four a chunk)
    int nslice;                       // slices of the fit's sums
    long long slice;                  // steps per slice
    size_t part_bytes, g_bytes, e_bytes;  // workspace: chunk partials, time-stage sums, phase table
};
DftPlan dft_plan(long long nt, int nz, int nw, int nk);
hipError_t launch_st_dft(const DftPlan &p, const double *x, long long nt, int nz, const double *zpos, double t0,
                         double w0, double dw, int nw, double k0, double dk, int nk, double *F, int *ridge,
                         void *work, hipStream_t st);
hipError_t launch_wave_fit(const double *x, long long nt, int nz, const double *zpos, double t0, double omega,
                           double *out, void *work, hipStream_t st);
// the allocation-free fit's static device scratch: its size, and its address on the
// current device (looked up once per device)
constexpr size_t kNoAllocScratchBytes = size_t(4) << 20;
hipError_t noalloc_scratch(void **ptr);
hipError_t launch_particle_signal(const double *ring, int ring_len, int ptot, int p_off, long long first,
                                  long long n, const int *start, const int *members, int n_layers, int component,
                                  double *x, hipStream_t st);
hipError_t launch_probe_signal(const double *ring, int ring_len, int nprobe, long long first, long long n,
                               int quantity, double *x, hipStream_t st);

} // namespace lbdem
