// Natural frequencies of the linearised mass-spring system (section "Natural Frequency
// Analysis": the generalised eigenproblem K v = w^2 M v).  Lanczos iterations on the
// symmetric operator A = M^-1/2 K M^-1/2 run on the device in FP64; the host takes the
// eigenvalues of the tridiagonal matrix they build (see cronos_natural_frequencies).
//
// K is the tangent stiffness of the Hookean springs of eq. (2) at the current positions:
// for a spring with unit direction n, length l and (actuated) rest length l0 its 3x3 block is
// k [n n^T + (1 - l0 / l)(I - n n^T)], entering the two diagonal blocks with + and the two
// off-diagonal blocks with -, so that df = -K dx; a mass below the contact plane adds the
// penalty stiffness k_g to its z diagonal.  Fixed masses are removed (their M^-1/2 is 0).
//
// Layout: the step's explicit incidence form (per-lane slices of (LDS slot, k, L0) with
// halo indices), one workgroup per block of masses whose positions and M^-1/2 q (with the
// halo's) are staged in LDS first; every sum is reduced in a fixed order, so a run is
// bitwise repeatable.
//
// A Lanczos step is two launches.  The vectors stay unnormalised, w_k = beta_{k-1} q_k: the apply
// kernel is linear, so it works on w_k while the previous launch's partial norms are still being
// summed, and scales its result by 1 / beta_{k-1} at the end; the update kernel scales what it
// reads.  (A separate normalisation was a third launch and another pass over the vector: 6.4 of
// 57.5 us per step on the 640,000-mass cantilever, 3.1 of 22 us on 11,520 masses.)
#include "kernels.h"

#include <mutex>
#include <vector>

// Workspace of cronos_natural_frequencies_noalloc (each GPU holds its own copy).  Host code
// never uses this name as an address: modes_scratch looks the device address up.
static __device__ __align__(256) double scratch[cronos::kModesScratchDoubles + cronos::kModesScratchExtra];

namespace cronos {
namespace {

constexpr int kMaxWaves = 16;
constexpr size_t kModesMaxLds = 150 * 1024;   // dynamic LDS of the staged apply kernel (of 160 KiB)
// workgroups and threads of the vector kernels of an iteration: every workgroup of the next kernel
// first sums these workgroups' partials, so there is one for each CU and no more
constexpr int kModesVecGroups = 256, kModesVecThreads = 512;

__device__ __forceinline__ double wave_add(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum over the workgroup: wavefront sums, then added in wavefront order by every thread (one
// barrier; `red` is not reused by the kernel).
__device__ __forceinline__ double workgroup_sum(double v, double* red) {
    v = wave_add(v);
    const int t = (int)threadIdx.x, nw = ((int)blockDim.x + 63) >> 6;
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w];
    return s;
}

// This thread's share of part[0..count): strided by the workgroup, the same in every workgroup.
__device__ __forceinline__ double own_parts(const double* __restrict__ part, int count) {
    double a = 0.0;
    for (int q = (int)threadIdx.x; q < count; q += (int)blockDim.x) a += part[q];
    return a;
}

// The norm of w_k: partials of the launch that wrote it, and where the first workgroup leaves
// beta_{k-1} and 1 / beta_{k-1} for the later kernels.
struct NormArgs {
    const double* __restrict__ part;
    int count;
    double* beta;
    double* inv;   // [2], by the parity of k
    int k;
};

// The sums over the workgroup of both arguments at once; returns 1 / beta_{k-1} from the first
// (a thread's own_parts of the norm) and leaves the second's sum in `other`.
__device__ __forceinline__ double norm_and_sum(const NormArgs& nm, double norm2, double& other, double* red) {
    norm2 = wave_add(norm2);
    other = wave_add(other);
    const int t = (int)threadIdx.x, nw = ((int)blockDim.x + 63) >> 6;
    if ((t & 63) == 0) {
        red[t >> 6] = norm2;
        red[kMaxWaves + (t >> 6)] = other;
    }
    __syncthreads();
    norm2 = other = 0.0;
    for (int w = 0; w < nw; ++w) {
        norm2 += red[w];
        other += red[kMaxWaves + w];
    }
    const double b = sqrt(norm2), inv = b > 0.0 ? 1.0 / b : 0.0;
    if (blockIdx.x == 0 && t == 0) {
        nm.inv[nm.k & 1] = inv;
        if (nm.k > 0) nm.beta[nm.k - 1] = b;
    }
    return inv;
}

__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// M^-1/2 per mass and a random start vector (zero on fixed masses); partial squared norms;
// zeros in q_prev (the Lanczos vector before the first, cleared here by a kernel rather than a
// memset node so that the sequence stays a plain kernel chain).
__global__ void __launch_bounds__(kModesVecThreads)
modes_init_kernel(const float4* __restrict__ x, const float* __restrict__ mass, double* __restrict__ ism,
                  double* __restrict__ w, double* __restrict__ q_prev, double* __restrict__ part,
                  double* __restrict__ inv, int n, unsigned long long seed) {
    __shared__ double red[kMaxWaves];
    double nn = 0.0;
    for (int i = (int)(blockIdx.x * blockDim.x + threadIdx.x); i < n; i += (int)(gridDim.x * blockDim.x)) {
        const bool free_mass = x[i].w != 0.0f;
        ism[i] = free_mass ? 1.0 / sqrt((double)mass[i]) : 0.0;
        for (int c = 0; c < 3; ++c) {
            const unsigned long long h = mix64(seed + 0x9e3779b97f4a7c15ull * (unsigned long long)(3 * (long long)i + c + 1));
            const double u = free_mass ? (double)(h >> 11) * 0x1.0p-53 - 0.5 : 0.0;
            w[3 * (long)i + c] = u;
            q_prev[3 * (long)i + c] = 0.0;
            nn += u * u;
        }
    }
    const double s = workgroup_sum(nn, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
    if (blockIdx.x == 0 && threadIdx.x == 0) inv[1] = 0.0;   // of the vector before the first
}

struct ApplyArgs {
    const float4* __restrict__ x;
    const double* __restrict__ ism;
    const int32_t* __restrict__ slice_ptr;
    const uint16_t* __restrict__ nbr;
    const float2* __restrict__ kl;
    const uint16_t* __restrict__ grp;
    const float* __restrict__ factor;
    const int32_t* __restrict__ halo_ptr;
    const int32_t* __restrict__ halo_idx;
    const uint16_t* __restrict__ lane_mass;
    int n, block, lds_slots;
    int ground;
    float ground_z, ground_k;
};

// 1/sqrt(s) to FP64 accuracy: the hardware estimate y (relative error 2^-24 at most) refined by
// one third-order step, y (1 + e/2 + 3 e^2 / 8) with e = 1 - s y^2, whose error is e^3: as close
// as two Newton steps in five operations instead of eight, and far cheaper than a correctly
// rounded square root followed by a division.
__device__ __forceinline__ double rsqrt_fp64(double s) {
    const double y = __builtin_amdgcn_rsq(s);
    const double e = __builtin_fma(-(s * y), y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// Contribution of spring (i, j) to (K u)_i: with d = x_j - x_i, l = |d| and v = u_i - u_j,
//   k [n n^T + (1 - l0/l)(I - n n^T)] v = (k - t) v + (t / l^2) (d . v) d,   t = k l0 / l
// (fused multiply-adds; 37 operations against 50 with n formed first).
__device__ __forceinline__ void spring_hessian(float4 xi, float4 xj, double u0, double u1, double u2, double v0,
                                               double v1, double v2, double kk, double l0, double& k0, double& k1,
                                               double& k2) {
    const double dx = (double)xj.x - (double)xi.x, dy = (double)xj.y - (double)xi.y, dz = (double)xj.z - (double)xi.z;
    const double il = rsqrt_fp64(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)));
    const double d0 = u0 - v0, d1 = u1 - v1, d2 = u2 - v2;
    const double t = kk * l0 * il, a = kk - t;
    const double p = t * (il * il) * __builtin_fma(dx, d0, __builtin_fma(dy, d1, dz * d2));
    k0 = __builtin_fma(p, dx, __builtin_fma(a, d0, k0));
    k1 = __builtin_fma(p, dy, __builtin_fma(a, d1, k1));
    k2 = __builtin_fma(p, dz, __builtin_fma(a, d2, k2));
}

// The end of an apply kernel for the mass's owning lane (`mine`): its (K u)_i in k0..k2, from the
// unnormalised w_k, becomes y = M^-1/2 K M^-1/2 q_k, and the workgroup's part of q_k . y.
__device__ __forceinline__ void finish_apply(const NormArgs& nm, double norm2, bool mine, int i, double si, double k0,
                                             double k1, double k2, const double* __restrict__ w,
                                             double* __restrict__ y, double* __restrict__ part, double* red) {
    const double y0 = si * k0, y1 = si * k1, y2 = si * k2;
    double dot = mine ? w[3 * (long)i] * y0 + w[3 * (long)i + 1] * y1 + w[3 * (long)i + 2] * y2 : 0.0;
    const double inv = norm_and_sum(nm, norm2, dot, red);
    if (mine) {
        y[3 * (long)i] = y0 * inv;
        y[3 * (long)i + 1] = y1 * inv;
        y[3 * (long)i + 2] = y2 * inv;
    }
    if (threadIdx.x == 0) part[blockIdx.x] = dot * inv * inv;
}

// y = A q with the workgroup's masses and halo staged in LDS: positions (float4) and
// u = M^-1/2 w (FP64) per slot, so the incidence loop reads no global memory but its entries.
// L lanes per mass (1 or 4): lane j of a mass takes incidence rows j, j + L, ... and the partial
// sums are combined by a fixed pairing of cross-lane exchanges.  The first rows' entries are
// loaded before the barrier.  A body below 131,072 masses leaves most SIMDs idle with one lane a
// mass, each lane then waiting 26 times for its next entry: 11,520 masses 14.9 -> 5.9 us.
template <int L>
__global__ void __launch_bounds__(1024) modes_apply_lds_kernel(ApplyArgs a, NormArgs nm, const double* __restrict__ w,
                                                               double* __restrict__ y, double* __restrict__ part) {
    extern __shared__ float4 sx[];                       // [lds_slots] positions
    double* su = reinterpret_cast<double*>(sx + a.lds_slots);   // [lds_slots][3] u
    __shared__ double red[2 * kMaxWaves];
    constexpr int B = L == 1 ? 4 : 8;   // rows whose entries are in flight together
    const int b = (int)blockIdx.x, t = (int)threadIdx.x, m = t / L, sub = t % L;
    const int base = b * a.block;
    const int own = a.lane_mass[base + m];
    const int i = base + own;
    const int s = __builtin_amdgcn_readfirstlane((base + m) >> 6);
    const int e0 = __builtin_amdgcn_readfirstlane(a.slice_ptr[s]);
    const int width = __builtin_amdgcn_readfirstlane((a.slice_ptr[s + 1] - e0) >> 6);
    const int rows = (width - sub + L - 1) / L;   // this lane's
    const int e = e0 + sub * 64 + (m & 63);       // its row r: 64 L r further
    int slot[B], grp[B];
    float kx[B], kl0[B];
    auto load = [&](int r0) {
#pragma unroll
        for (int u = 0; u < B; ++u) {
            slot[u] = own;   // a missing row is skipped like the padding
            grp[u] = 0;
            if (r0 + u < rows) {
                const int q = e + (r0 + u) * (64 * L);
                slot[u] = a.nbr[q];
                const float2 c = a.kl[q];
                kx[u] = c.x;
                kl0[u] = c.y;
                if (a.grp) grp[u] = a.grp[q];
            }
        }
    };
    load(0);
    const double norm2 = own_parts(nm.part, nm.count);
    const int h0 = a.halo_ptr[b], slots = a.block + (a.halo_ptr[b + 1] - h0);
    for (int sl = t; sl < slots; sl += (int)blockDim.x) {
        const int j = sl < a.block ? base + sl : a.halo_idx[h0 + sl - a.block];
        float4 xm = make_float4(0.f, 0.f, 0.f, 0.f);
        double u0 = 0.0, u1 = 0.0, u2 = 0.0;
        if (j < a.n) {
            xm = a.x[j];
            const double sm = a.ism[j];
            u0 = sm * w[3 * (long)j];
            u1 = sm * w[3 * (long)j + 1];
            u2 = sm * w[3 * (long)j + 2];
        }
        sx[sl] = xm;
        su[3 * sl] = u0;
        su[3 * sl + 1] = u1;
        su[3 * sl + 2] = u2;
    }
    __syncthreads();
    const float4 xi = sx[own];
    const double u0 = su[3 * own], u1 = su[3 * own + 1], u2 = su[3 * own + 2];
    double k0 = 0.0, k1 = 0.0, k2 = 0.0;
    for (int r0 = 0;;) {
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (slot[u] == own) continue;  // padding
            double l0 = (double)kl0[u];
            if (a.grp) l0 *= (double)a.factor[grp[u]];
            const int sl = slot[u];
            spring_hessian(xi, sx[sl], u0, u1, u2, su[3 * sl], su[3 * sl + 1], su[3 * sl + 2], (double)kx[u], l0, k0, k1,
                           k2);
        }
        r0 += B;
        if (r0 * L >= width) break;
        load(r0);
    }
#pragma unroll
    for (int o = 1; o < L; o <<= 1) {
        k0 += __shfl_xor(k0, o, 64);
        k1 += __shfl_xor(k1, o, 64);
        k2 += __shfl_xor(k2, o, 64);
    }
    const bool mine = sub == 0 && i < a.n;
    if (a.ground && xi.z < a.ground_z) k2 += (double)a.ground_k * u2;
    finish_apply(nm, norm2, mine, i, mine ? a.ism[i] : 0.0, k0, k1, k2, w, y, part, red);
}

// y = A q for a full box in the structured-box layout (512 masses per aligned 8 x 8 x 8 Morton
// cube, every mass linked to its 26 grid neighbours, as the step's structured-box form): the
// cube and its one-node halo are staged as a 10 x 10 x 10 tile of positions and u = M^-1/2 w,
// each neighbour sits at a fixed tile offset, k comes from the table per (boundary class,
// direction) - or, where a whole wavefront is interior, per direction kind - and L0 per
// direction kind, so no incidence data is read.  Halo cells outside the box hold a far position
// and u = 0 with k = 0: no contribution.
struct GridApplyArgs {
    const float4* __restrict__ x;
    const double* __restrict__ ism;
    const int32_t* __restrict__ halo;   // [nblk][488] new index of each halo cell, -1 outside
    const int4* __restrict__ org;       // [nblk] grid coordinates of the block's first node
    const float* __restrict__ kcls;     // [27][26] k per (boundary class, direction)
    const uint32_t* __restrict__ tab;   // [512] lane's tile cell | lx << 10 | ly << 13 | lz << 16,
                                        // then [488] tile cell of each halo slot
    int nblk;
    int nx, ny, nz;
    float kin[3];                       // interior k per direction kind
    float l0[3];                        // rest length per direction kind (1, 2, 3 non-zero offsets)
    int ground;
    float ground_z, ground_k;
};

constexpr int kTilePitch = 10, kTilePlane = 100, kTileHalo = 488, kTileMasses = 512;

template <bool INTERIOR>
__device__ __forceinline__ void grid_hessian(const float4* __restrict__ tx, const double* __restrict__ tu,
                                             const float* __restrict__ kc, const GridApplyArgs& a, int cell, float4 xi,
                                             double u0, double u1, double u2, double& k0, double& k1, double& k2) {
#pragma unroll
    for (int d = 0; d < 26; ++d) {
        const int e = d < 13 ? d : d + 1;   // the 3 x 3 x 3 stencil without its centre, (dz, dy, dx) order
        const int ox = e % 3 - 1, oy = (e / 3) % 3 - 1, oz = e / 9 - 1;
        const int kind = (ox != 0) + (oy != 0) + (oz != 0) - 1;
        const int nc = cell + (oz * kTilePitch + oy) * kTilePitch + ox;
        spring_hessian(xi, tx[nc], u0, u1, u2, tu[3 * nc], tu[3 * nc + 1], tu[3 * nc + 2],
                       (double)(INTERIOR ? a.kin[kind] : kc[d]), (double)a.l0[kind], k0, k1, k2);
    }
}

// PARTS workgroups per cube (1 or 2, halves in z: planes 0-3 and 4-7).  Halves stage 600 cells for
// 256 masses instead of 1000 for 512, but fill the last round of a launch better (see
// modes_grid_parts).
template <int PARTS>
__global__ void __launch_bounds__(kTileMasses / PARTS)
modes_apply_grid_kernel(GridApplyArgs a, NormArgs nm, const double* __restrict__ w, double* __restrict__ y,
                        double* __restrict__ part) {
    constexpr int T = kTileMasses / PARTS, PLANES = 8 / PARTS + 2;
    __shared__ float4 tx[PLANES * kTilePlane];
    __shared__ double tu[3 * PLANES * kTilePlane];
    __shared__ float kc[27 * 26];
    __shared__ double red[2 * kMaxWaves];
    // each of the 8 XCDs takes a contiguous eighth of the cubes, whose halos then meet in its L2
    const int per = (a.nblk * PARTS + 7) >> 3;
    const int bb = (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
    const int t = (int)threadIdx.x;
    if (bb >= a.nblk * PARTS) {   // the grid is rounded up to a multiple of 8
        if (t == 0) part[blockIdx.x] = 0.0;
        return;
    }
    const int b = bb / PARTS, z0 = bb % PARTS * (8 / PARTS);   // first tile plane staged
    const int i = b * kTileMasses + bb % PARTS * T + t;   // the box holds whole cubes: i < n
    const uint32_t info = a.tab[i - b * kTileMasses];
    const int cell = (int)(info & 1023u) - z0 * kTilePlane;
    auto stage = [&](int c, int g) {
        float4 xm = make_float4(1e18f, 1e18f, 1e18f, 0.0f);
        double u0 = 0.0, u1 = 0.0, u2 = 0.0;
        if (g >= 0) {
            const double sm = a.ism[g];
            xm = a.x[g];
            u0 = sm * w[3 * (long)g + 0];
            u1 = sm * w[3 * (long)g + 1];
            u2 = sm * w[3 * (long)g + 2];
        }
        tx[c] = xm;
        tu[3 * c + 0] = u0;
        tu[3 * c + 1] = u1;
        tu[3 * c + 2] = u2;
    };
    stage(cell, i);
    if (PARTS == 2 && t < 64) {
        // the other half's plane next to this one (lz = 4 or 3): x and y from the bits of t
        const int z = z0 ? 0x24 : 0x100;   // lz's bits (2, 5, 8) of mass index: 3 or 4
        const int m = (t & 3) | (t >> 2 & 3) << 3 | (t >> 4 & 3) << 6 | z;
        stage((int)(a.tab[m] & 1023u) - z0 * kTilePlane, b * kTileMasses + m);
    }
    for (int h = t; h < kTileHalo; h += T) {
        const int c = (int)a.tab[kTileMasses + h] - z0 * kTilePlane;
        if (PARTS == 1 || (c >= 0 && c < PLANES * kTilePlane)) stage(c, a.halo[(long)b * kTileHalo + h]);
    }
    const double norm2 = own_parts(nm.part, nm.count);
    const int4 o = a.org[b];
    const bool face = o.x == 0 || o.y == 0 || o.z == 0 || o.x + 8 >= a.nx || o.y + 8 >= a.ny || o.z + 8 >= a.nz;
    int cls = 13;
    if (face) {
        for (int r = t; r < 27 * 26; r += T) kc[r] = a.kcls[r];
        const int gx = o.x + (int)((info >> 10) & 7u), gy = o.y + (int)((info >> 13) & 7u),
                  gz = o.z + (int)((info >> 16) & 7u);
        cls = (gx == 0 ? 0 : gx == a.nx - 1 ? 2 : 1) + 3 * (gy == 0 ? 0 : gy == a.ny - 1 ? 2 : 1) +
              9 * (gz == 0 ? 0 : gz == a.nz - 1 ? 2 : 1);
    }
    __syncthreads();
    const float4 xi = tx[cell];
    const double u0 = tu[3 * cell + 0], u1 = tu[3 * cell + 1], u2 = tu[3 * cell + 2];
    double k0 = 0.0, k1 = 0.0, k2 = 0.0;
    if (__builtin_amdgcn_ballot_w64(cls != 13) == 0)
        grid_hessian<true>(tx, tu, kc, a, cell, xi, u0, u1, u2, k0, k1, k2);
    else
        grid_hessian<false>(tx, tu, kc + 26 * cls, a, cell, xi, u0, u1, u2, k0, k1, k2);
    if (a.ground && xi.z < a.ground_z) k2 += (double)a.ground_k * u2;
    finish_apply(nm, norm2, true, i, a.ism[i], k0, k1, k2, w, y, part, red);
}

// y = A q for the masses of workgroup-block b, and the block's part of q . y; neighbours read
// from global memory (used when the staged form's LDS would not fit).
__global__ void __launch_bounds__(1024) modes_apply_kernel(ApplyArgs a, NormArgs nm, const double* __restrict__ w,
                                                           double* __restrict__ y, double* __restrict__ part) {
    __shared__ double red[2 * kMaxWaves];
    const int b = (int)blockIdx.x, t = (int)threadIdx.x;
    const int base = b * a.block;
    const int i = base + a.lane_mass[base + t];
    const double norm2 = own_parts(nm.part, nm.count);
    double k0 = 0.0, k1 = 0.0, k2 = 0.0, si = 0.0;
    if (i < a.n) {
        const float4 xi = a.x[i];
        si = a.ism[i];
        const double u0 = si * w[3 * (long)i], u1 = si * w[3 * (long)i + 1], u2 = si * w[3 * (long)i + 2];
        const int s = (base + t) >> 6, lane = t & 63;
        const int e0 = a.slice_ptr[s];
        const int width = (a.slice_ptr[s + 1] - e0) >> 6;
        const int h0 = a.halo_ptr[b];
        for (int r = 0, e = e0 + lane; r < width; ++r, e += 64) {
            const int slot = a.nbr[e];
            const int j = slot < a.block ? base + slot : a.halo_idx[h0 + slot - a.block];
            if (j == i) continue;  // padding
            const float2 c = a.kl[e];
            double l0 = (double)c.y;
            if (a.grp) l0 *= (double)a.factor[a.grp[e]];
            const double sj = a.ism[j];
            spring_hessian(xi, a.x[j], u0, u1, u2, sj * w[3 * (long)j], sj * w[3 * (long)j + 1], sj * w[3 * (long)j + 2],
                           (double)c.x, l0, k0, k1, k2);
        }
        if (a.ground && xi.z < a.ground_z) k2 += (double)a.ground_k * u2;
    }
    finish_apply(nm, norm2, i < a.n, i, si, k0, k1, k2, w, y, part, red);
}

// alpha_k = q_k . y (from the apply kernel's parts); w_{k+1} = y - alpha_k q_k - beta_{k-1} q_{k-1}
// written over w_{k-1}; partial squared norms of w_{k+1}.  Memory-bound: 24 B read and 8 written
// per component, two components a load.
__global__ void __launch_bounds__(kModesVecThreads)
modes_update_kernel(const double* __restrict__ apart, int n_apart, const double* __restrict__ y,
                    const double* __restrict__ w, double* __restrict__ wp, const double* __restrict__ inv,
                    double* __restrict__ alpha, const double* __restrict__ beta, int k, double* __restrict__ part,
                    long n3) {
    __shared__ double red[kMaxWaves], red2[kMaxWaves];
    const double ik = inv[k & 1], ip = inv[(k & 1) ^ 1];
    const double bp = k > 0 ? beta[k - 1] : 0.0;
    const double al = workgroup_sum(own_parts(apart, n_apart), red);
    double nn = 0.0;
    auto one = [&](double yv, double wv, double pv) {
        const double r = __builtin_fma(-bp, pv * ip, __builtin_fma(-al, wv * ik, yv));
        nn = __builtin_fma(r, r, nn);
        return r;
    };
    const long step = (long)gridDim.x * blockDim.x, first = (long)blockIdx.x * blockDim.x + threadIdx.x;
    for (long q = first; q < n3 / 2; q += step) {
        const double2 yv = reinterpret_cast<const double2*>(y)[q], wv = reinterpret_cast<const double2*>(w)[q];
        double2 pv = reinterpret_cast<double2*>(wp)[q];
        pv.x = one(yv.x, wv.x, pv.x);
        pv.y = one(yv.y, wv.y, pv.y);
        reinterpret_cast<double2*>(wp)[q] = pv;
    }
    if (first == 0 && (n3 & 1)) wp[n3 - 1] = one(y[n3 - 1], w[n3 - 1], wp[n3 - 1]);
    const double s = workgroup_sum(nn, red2);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
    if (blockIdx.x == 0 && threadIdx.x == 0) alpha[k] = al;
}

// beta_{k-1} = |w_k| alone, summed as the apply kernel of step k sums it (the same threads).
__global__ void __launch_bounds__(1024) modes_beta_kernel(NormArgs nm) {
    __shared__ double red[2 * kMaxWaves];
    double none = 0.0;
    (void)norm_and_sum(nm, own_parts(nm.part, nm.count), none, red);
}

}  // namespace

namespace {

int vec_groups(const DeviceArrays& d) {
    return (int)std::min<int64_t>((d.n + kModesVecThreads - 1) / kModesVecThreads, kModesVecGroups);
}

size_t staged_lds(const DeviceArrays& d) { return (size_t)d.lds_slots * (sizeof(float4) + 3 * sizeof(double)); }

// Lanes per mass of the staged general operator.  Four where one lane a mass would leave most of
// the chip's 1024 SIMDs with less than two wavefronts (below 131,072 masses, the line at which the
// step's own default changes) and the workgroup has room for them.  Measured, 1 against 4 lanes:
// 11,520 masses 14.9 / 5.9 us; 62,073 masses (128-mass workgroups) 17.5 / 12.0 us.
int apply_lanes(const DeviceArrays& d) { return d.n < 131072 && d.block * 4 <= 1024 ? 4 : 1; }

// Workgroups per cube of the structured-box operator.  A CU works through its workgroups' FP64
// arithmetic at a fixed rate, so a launch takes as long as the CU with the most of it: halves are
// taken where they cut that maximum by a fifth or more, since each half stages 1.2 times its share.
int grid_parts(const DeviceArrays& d, int cus) {
    const int64_t whole = 2 * ((d.nblk + cus - 1) / cus), halves = (2 * d.nblk + cus - 1) / cus;
    return 5 * halves <= 4 * whole ? 2 : 1;
}

unsigned grid_groups(const DeviceArrays& d, int cus) {
    return (unsigned)((d.nblk * grid_parts(d, cus) + 7) / 8 * 8);
}

// Threads of an apply workgroup.
int apply_threads(const DeviceArrays& d, int cus) {
    if (d.grid) return kTileMasses / grid_parts(d, cus);
    return staged_lds(d) <= kModesMaxLds ? d.block * apply_lanes(d) : d.block;
}

}  // namespace

int64_t modes_apply_parts(const DeviceArrays& d) { return d.grid ? (2 * d.nblk + 7) / 8 * 8 : d.nblk; }

hipError_t launch_modes_init(const DeviceArrays& d, int cur, ModesBuffers& m, unsigned long long seed, hipStream_t st) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&m.cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(modes_init_kernel, dim3(vec_groups(d)), dim3(kModesVecThreads), 0, st, d.x[cur], d.mass, m.ism,
                       m.q[1], m.q[0], m.part_u, m.inv, (int)d.n, seed);
    return hipGetLastError();
}

hipError_t launch_modes_iteration(const DeviceArrays& d, int cur, const StepParams& p, ModesBuffers& m, int k,
                                  hipStream_t st) {
    const double* w = m.q[(k + 1) & 1];   // w_k (the start vector sits in q[1])
    double* wp = m.q[k & 1];              // w_{k-1} in, w_{k+1} out
    const NormArgs nm{m.part_u, vec_groups(d), m.beta, m.inv, k};
    int parts = (int)d.nblk;
    if (d.grid) {
        const GridApplyArgs ga{d.x[cur], m.ism, d.grid_halo, d.grid_org, d.grid_k, d.grid_tab, (int)d.nblk,
                               d.grid_dim[0], d.grid_dim[1], d.grid_dim[2],
                               {d.grid_kin[0], d.grid_kin[1], d.grid_kin[2]},
                               {d.grid_l0[0], d.grid_l0[1], d.grid_l0[2]}, p.ground, p.ground_z, p.ground_k};
        const dim3 g(grid_groups(d, m.cus)), th((unsigned)apply_threads(d, m.cus));
        parts = (int)g.x;
        if (grid_parts(d, m.cus) == 2) hipLaunchKernelGGL(modes_apply_grid_kernel<2>, g, th, 0, st, ga, nm, w, m.y, m.part_a);
        else hipLaunchKernelGGL(modes_apply_grid_kernel<1>, g, th, 0, st, ga, nm, w, m.y, m.part_a);
    } else {
        const ApplyArgs a{d.x[cur], m.ism, d.slice_ptr, d.nbr, d.kl, d.grp, d.factor, d.halo_ptr, d.halo_idx,
                          d.lane_mass, (int)d.n, d.block, d.lds_slots, p.ground, p.ground_z, p.ground_k};
        const size_t lds = staged_lds(d);
        const dim3 g((unsigned)d.nblk), th((unsigned)apply_threads(d, m.cus));
        if (lds > kModesMaxLds) hipLaunchKernelGGL(modes_apply_kernel, g, th, 0, st, a, nm, w, m.y, m.part_a);
        else if (apply_lanes(d) == 4) hipLaunchKernelGGL(modes_apply_lds_kernel<4>, g, th, lds, st, a, nm, w, m.y, m.part_a);
        else hipLaunchKernelGGL(modes_apply_lds_kernel<1>, g, th, lds, st, a, nm, w, m.y, m.part_a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(modes_update_kernel, dim3(vec_groups(d)), dim3(kModesVecThreads), 0, st, m.part_a, parts, m.y, w,
                       wp, m.inv, m.alpha, m.beta, k, m.part_u, 3 * (long)d.n);
    return hipGetLastError();
}

hipError_t launch_modes_beta(const DeviceArrays& d, ModesBuffers& m, int k, hipStream_t st) {
    const NormArgs nm{m.part_u, vec_groups(d), m.beta, m.inv, k};
    hipLaunchKernelGGL(modes_beta_kernel, dim3(1), dim3((unsigned)apply_threads(d, m.cus)), 0, st, nm);
    return hipGetLastError();
}

hipError_t modes_scratch(int device, double** ptr) {
    static std::mutex mu;
    static std::vector<double*> addr;   // per device ordinal
    std::lock_guard<std::mutex> lock(mu);
    if (device < 0) return hipErrorInvalidDevice;
    if ((int)addr.size() <= device) addr.resize(device + 1, nullptr);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = static_cast<double*>(p);
    }
    *ptr = addr[device];
    return hipSuccess;
}

}  // namespace cronos
