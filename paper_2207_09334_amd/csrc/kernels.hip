// Device kernels of the mass-spring step for gfx950 (CDNA4, wave64).
//
// One time step is one launch of `step_kernel` (actuated bodies in the compact table forms
// compute their actuation factors inside it; the explicit form takes a separate actuation
// launch).  It fuses what Algorithm 1 splits into a spring pass and a mass pass: every lane
// owns one mass (or lanes share one: `step_lanes_kernel`, `step_quads_kernel`), walks that mass's incidence
// list in a fixed order and sums the eq. (2) spring forces itself, so no force is ever written
// twice and no atomic is needed; the sum is bitwise reproducible run to run.
//
// Memory: positions are float4 (x, y, z, 1/m) so one 16-byte load fetches a neighbour; a
// workgroup first copies its own masses and its halo (the neighbours outside the workgroup)
// into LDS, then every incidence reads its neighbour from LDS.  The incidence stream is laid
// out column-major per 64-mass slice, so each wavefront's loads are contiguous; in the compact
// forms an entry is one 16-bit word (passive bodies: neighbour slot and index into the LDS
// table of distinct (k, L0) pairs) or one 32-bit word (also the actuation factor).
// Workgroups are spread so that each of the 8 XCDs gets a contiguous range of the Morton
// order (their halos then overlap within one L2).  A workgroup's lanes take its masses in
// order of decreasing degree; where the step streams from HBM (actuated 32-bit form beyond the
// Infinity Cache) a variant reads the velocities and writes the new state through LDS in mass
// order instead of where each lane's mass lies.
//
// A full box of masses linked to all 26 grid neighbours takes `step_grid_kernel` instead: one
// 512-thread workgroup per aligned 8 x 8 x 8 cube stages the cube and its one-node halo as a
// 10 x 10 x 10 tile and reads each neighbour at a fixed tile offset, with no incidence data.
//
// Precision: FP32 state and FP32 accumulation.  The elongation |d| - L0 of a nearly relaxed
// spring is a difference of nearly equal numbers; it is computed as (|d|^2 - L0^2)/(|d| + L0)
// with |d|^2 - L0^2 formed in FP64 from the FP32 differences (exact squares, L0^2 held
// exactly), so its error is about an ulp of the elongation itself, not of L0.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace cronos {

namespace {

__device__ __forceinline__ int logical_block(int nblk) {
    const int per = (nblk + 7) >> 3;
    return (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
}

// Coordinate-difference modes of the spring arithmetic (see hooke_fac).
enum : int { kPlain = 0, kExactZ = 1, kExactAll = 2 };

// Added to |d|^2 as it is summed (an FP64 addend far below half an ulp of any real spring's, so no
// bit of those changes): keeps a zero-length spring's denominator above zero, and its factor
// finite, without an instruction of its own.
constexpr double kLengthFloor = 1e-37;

// e^2 + kLengthFloor in one instruction: left to itself the compiler copies the constant into the
// accumulator of a two-address multiply-add first (two more instructions per spring).  A loop around it
// is not unrolled by the compiler, which may not copy such an instruction.
__device__ __forceinline__ double square_above_floor(double e) {
    double s;
    asm("v_fma_f64 %0, %1, %1, %2" : "=v"(s) : "v"(e), "s"(kLengthFloor));
    return s;
}

// Scalar factor of the Hooke force of eq. (2) for the spring from (xi, yi, zi) to (xj, yj, zj):
// the force on the first end is fac * d with d = xj - xi; a zero-length spring gives 0 (its d
// is 0 and fac stays finite).  Every step below is unchanged, bit for bit, when d changes sign,
// so both ends of a spring see the same factor.
//
// Elongation: |d| - L0 = (|d|^2 - L0^2) / (|d| + L0).  The numerator is formed in FP64 from the
// FP32 differences: the square of a 24-bit value is exact in 53 bits, L0^2 (q) is held exactly,
// so near rest the cancellation in |d|^2 - L0^2 loses nothing that matters (the error is
// ~1e-16 of L0^2, against FP32's ~6e-8).  On this chip an FP64 FMA takes the issue slot of an
// FP32 one, so five FP64 operations replace the twenty-odd FP32 ones of an error-free FP32
// formulation.
// EX: d = xj - xi is exact in FP32 whenever the two coordinates are within a factor of two of
// each other (Sterbenz); near a coordinate plane it is not, and for a nearly relaxed spring
// that one-ulp error in d would be a large fraction of the elongation.  kExactAll takes the
// differences in FP64 (exact for any two FP32 values of similar scale), so the elongation is
// that of the stored positions whatever their magnitude; kExactZ does so for z only, for
// wavefronts near the z = 0 plane alone (the contact plane); kPlain widens the FP32 ones.
template <int EX>
__device__ __forceinline__ float hooke_fac(float xi, float yi, float zi, float xj, float yj, float zj, float k,
                                           float l0, double q, float& dx, float& dy, float& dz) {
    dx = xj - xi;
    dy = yj - yi;
    dz = zj - zi;
    double ex = dx, ey = dy, ez = dz;
    if (EX == kExactAll) {
        ex = (double)xj - (double)xi;
        ey = (double)yj - (double)yi;
    }
    if (EX != kPlain) ez = (double)zj - (double)zi;
    const double s = __builtin_fma(ex, ex, __builtin_fma(ey, ey, square_above_floor(ez)));
    const float diff = (float)(s - q);
    const float s2 = (float)s;
    const float len = __builtin_amdgcn_sqrtf(s2);
    // |d| (|d| + L0) = s2 + L0 |d| to within an ulp
    const float den = __builtin_fmaf(l0, len, s2);
    return k * diff * __builtin_amdgcn_rcpf(den);
}

// The same with L0^2 formed here (exact in FP64).
template <int EX>
__device__ __forceinline__ float hooke_fac(float xi, float yi, float zi, float xj, float yj, float zj, float k,
                                           float l0, float& dx, float& dy, float& dz) {
    return hooke_fac<EX>(xi, yi, zi, xj, yj, zj, k, l0, (double)l0 * (double)l0, dx, dy, dz);
}

// Hooke force of eq. (2) on mass i from one spring to a neighbour at (xj, yj, zj),
// accumulated into f.
template <int EX>
__device__ __forceinline__ void hooke(float xi, float yi, float zi, float xj, float yj, float zj,
                                      float k, float l0, float& fx, float& fy, float& fz) {
    float dx, dy, dz;
    const float fac = hooke_fac<EX>(xi, yi, zi, xj, yj, zj, k, l0, dx, dy, dz);
    fx = __builtin_fmaf(fac, dx, fx);
    fy = __builtin_fmaf(fac, dy, fy);
    fz = __builtin_fmaf(fac, dz, fz);
}

// L0^2 of a parameter-table entry c = (k, L0, L0^2 as an FP64 value in its last two words).
__device__ __forceinline__ double table_l0sq(float4 c) {
    const unsigned long long bits =
        ((unsigned long long)__float_as_uint(c.w) << 32) | (unsigned long long)__float_as_uint(c.z);
    return __longlong_as_double((long long)bits);
}

// The same with a parameter-table entry c = (k, L0, L0^2 in FP64); an actuated spring scales L0
// by its factor g and squares it here.
template <bool ACT, int EX>
__device__ __forceinline__ float hooke_fac_tab(float4 xi, float4 xj, float4 c, float g, float& dx, float& dy,
                                               float& dz) {
    if (ACT) return hooke_fac<EX>(xi.x, xi.y, xi.z, xj.x, xj.y, xj.z, c.x, c.y * g, dx, dy, dz);
    return hooke_fac<EX>(xi.x, xi.y, xi.z, xj.x, xj.y, xj.z, c.x, c.y, table_l0sq(c), dx, dy, dz);
}

// Stage the workgroup's masses (in mass order) and its halo in LDS; returns the block-relative
// index of the mass this lane owns (lanes take the block's masses by decreasing degree).
__device__ __forceinline__ int stage_positions(float4* __restrict__ sx, const float4* __restrict__ xin,
                                               const int32_t* __restrict__ halo_ptr,
                                               const int32_t* __restrict__ halo_idx,
                                               const uint16_t* __restrict__ lane_mass, int b, int base, int n,
                                               int block) {
    const int t = threadIdx.x;
    const int own = lane_mass[base + t];
    float4 xt = make_float4(0.f, 0.f, 0.f, 0.f);
    if (base + t < n) xt = xin[base + t];
    sx[t] = xt;
    const int h0 = halo_ptr[b], h1 = halo_ptr[b + 1];
    for (int h = h0 + t; h < h1; h += block) sx[block + (h - h0)] = xin[halo_idx[h]];
    __syncthreads();
    return own;
}

template <int EX, int BATCH>
constexpr int kPart = EX == kExactAll && BATCH > 2 ? BATCH / 2 : BATCH;

// A lane's entries, row after row of its slice (64 masses; the slice, and so the trip count, is
// uniform across the wavefront), BATCH rows at a time: each batch is loaded while the one before
// it is worked on, and the first before the workgroup's positions are staged, since entries depend
// on nothing in LDS.  A step waits on memory more than it computes, and a slice's five to ten
// batches were one full latency each when loaded as they were needed: a population of 64 robots
// (337,000 masses) 13.2 -> 11.4 us a step; the cantilever by 16-bit entries 18.3 -> 17.1, by 32-bit
// ones 19.7 -> 18.3; the quadruped with one lane per mass 7.7 -> 6.8.
// The springs are added in row order whatever BATCH is.
template <class Rows, int BATCH>
struct RowWalk {
    Rows rows;
    int w = 0;   // rows of the slice
    typename Rows::Item q[BATCH];

    // the first batch; rows past the slice's end are the next slice's or the arrays' padding
    // (kEntryPad), and never used
    __device__ __forceinline__ void start(int s, int nslice, const int32_t* __restrict__ slice_ptr) {
        s = __builtin_amdgcn_readfirstlane(s);
        if (s >= nslice) return;
        const int e0 = __builtin_amdgcn_readfirstlane(slice_ptr[s]);
        w = __builtin_amdgcn_readfirstlane((slice_ptr[s + 1] - e0) >> 6);
        rows.at(e0 + (int)(threadIdx.x & 63u), w);
        if (w > 0) fetch(0);
    }
    __device__ __forceinline__ void fetch(int r) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) q[u] = rows.load(r + u);
    }
    // one(item) for every row.  PART: rows whose LDS reads may be in flight together (the
    // exact-difference loop holds more live values per row; half as many keep its registers, and
    // so its occupancy, those of the plain one)
    template <int PART, class One>
    __device__ __forceinline__ void run(One one) {
        int r = 0;
        for (; r + BATCH <= w; r += BATCH) {
            typename Rows::Item c[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) c[u] = q[u];
            if (r + BATCH < w) fetch(r + BATCH);
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                one(c[u]);
                if (PART < BATCH && (u + 1) % PART == 0) __builtin_amdgcn_sched_barrier(0);
            }
        }
        tail<0, BATCH>(w - r, one);
    }
    // the last `left` < N rows, q[BASE ...], in straight runs of 4, 2 and 1
    template <int BASE, int N, class One>
    __device__ __forceinline__ void tail(int left, One one) {
        if constexpr (N > 1) {
            constexpr int H = N / 2;
            if (left >= H) {
#pragma unroll
                for (int u = 0; u < H; ++u) one(q[BASE + u]);
                tail<BASE + H, H>(left - H, one);
            } else {
                tail<BASE, H>(left, one);
            }
        }
    }
};

// Sum of the spring forces on this lane's mass over its slice entries.  The slice (and so the
// trip count) is uniform across the wavefront; entries are fetched in batches of BATCH so
// that several loads are in flight before the first is consumed.
// (Loading a batch ahead as RowWalk does, three registers a row here, lost: the cantilever's 640,000 masses
// 30.8 -> 31.5 us, the quadruped 7.9 -> 8.7.)
template <bool ACT, int EX, int BATCH>
__device__ __forceinline__ void gather(const float4* __restrict__ sx, float4 xi, int s, int nslice,
                                       const int32_t* __restrict__ slice_ptr,
                                       const uint16_t* __restrict__ nbr, const float2* __restrict__ kl,
                                       const uint16_t* __restrict__ grp, const float* __restrict__ factor,
                                       float& fx, float& fy, float& fz) {
    fx = fy = fz = 0.0f;
    s = __builtin_amdgcn_readfirstlane(s);
    if (s >= nslice) return;
    const int lane = threadIdx.x & 63;
    const int e0 = __builtin_amdgcn_readfirstlane(slice_ptr[s]);
    const int w = __builtin_amdgcn_readfirstlane((slice_ptr[s + 1] - e0) >> 6);
    const uint16_t* pn = nbr + e0 + lane;
    const float2* pk = kl + e0 + lane;
    const uint16_t* pg = ACT ? grp + e0 + lane : nullptr;
    int r = 0;
    for (; r + BATCH <= w; r += BATCH) {
        int slot[BATCH];
        float2 c[BATCH];
        float f[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            slot[u] = pn[(r + u) * 64];
            c[u] = pk[(r + u) * 64];
            if (ACT) f[u] = factor[pg[(r + u) * 64]];
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const float4 xj = sx[slot[u]];
            const float l0 = ACT ? c[u].y * f[u] : c[u].y;
            hooke<EX>(xi.x, xi.y, xi.z, xj.x, xj.y, xj.z, c[u].x, l0, fx, fy, fz);
        }
    }
    for (; r < w; ++r) {
        const int slot = pn[r * 64];
        const float2 c = pk[r * 64];
        const float l0 = ACT ? c.y * factor[pg[r * 64]] : c.y;
        const float4 xj = sx[slot];
        hooke<EX>(xi.x, xi.y, xi.z, xj.x, xj.y, xj.z, c.x, l0, fx, fy, fz);
    }
}

// LDS read at a byte address.  The step kernels declare no static LDS, so their dynamic LDS
// (positions first) starts at address 0 (checked on the host) and an entry word can carry
// ready-made byte addresses.
typedef float lds_vec4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ lds_vec4 lds_v4(uint32_t byte) {
    return *(const __attribute__((address_space(3))) lds_vec4*)(size_t)byte;
}
__device__ __forceinline__ float4 lds_f4(uint32_t byte) {
    const lds_vec4 v = lds_v4(byte);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float lds_f1(uint32_t byte) {
    return *(const __attribute__((address_space(3))) float*)(size_t)byte;
}

// The same sum over the compact entry stream: one 32-bit word per entry and the parameter
// table of the simulation's distinct (k, L0) pairs staged in LDS at byte address T (a
// multiple of 8192, so "| T" adds it).
//   passive simulations: neighbour slot << 19 | pair index << 4, so the neighbour's byte
//     address is q >> 15 and the pair's is (q & 0x1FF0) | T;
//   actuated simulations: neighbour slot (bits 0-12) | pair index (bits 13-21) | index of
//     the spring's actuation factor in the workgroup's slice of the factor table, staged in
//     LDS at sf (bits 22-31, 0 = passive).
constexpr uint32_t kSlotBits = 13, kTypeBits = 9;

template <bool ACT>
__device__ __forceinline__ void decode_entry(uint32_t q, uint32_t tbase, uint32_t& xa, uint32_t& ca, uint32_t& g) {
    if (ACT) {
        xa = (q & ((1u << kSlotBits) - 1u)) << 4;
        ca = ((q >> (kSlotBits - 4)) & (((1u << kTypeBits) - 1u) << 4)) | tbase;
        g = q >> (kSlotBits + kTypeBits);
    } else {
        xa = q >> 15;
        ca = (q & (((1u << kTypeBits) - 1u) << 4)) | tbase;
        g = 0;
    }
}

template <class T>
struct CompactRows {
    const T* __restrict__ words;
    typedef uint32_t Item;
    __device__ __forceinline__ void at(int e, int) { words += e; }
    __device__ __forceinline__ Item load(int r) const { return (uint32_t)words[r * 64]; }
};

// The same over entries held in LDS, which has no padding: rows past the end repeat the last one.
struct ResidentRows {
    const uint32_t* words;
    int last;
    typedef uint32_t Item;
    __device__ __forceinline__ void at(int e, int w) {
        words += e;
        last = w - 1;
    }
    __device__ __forceinline__ Item load(int r) const { return words[min(r, last) * 64]; }
};

template <bool ACT, int EX, int BATCH, class Rows>
__device__ __forceinline__ void gather_table(uint32_t tbase, const float* __restrict__ sf, float4 xi,
                                             RowWalk<Rows, BATCH>& walk, float& fx, float& fy,
                                             float& fz) {
    fx = fy = fz = 0.0f;
    walk.template run<kPart<EX, BATCH>>([&](uint32_t q) {
        uint32_t xa, ca, gi;
        decode_entry<ACT>(q, tbase, xa, ca, gi);
        const float4 xj = lds_f4(xa);
        const float4 c = lds_f4(ca);
        const float g = ACT ? sf[gi] : 1.0f;
        float dx, dy, dz;
        const float fac = hooke_fac_tab<ACT, EX>(xi, xj, c, g, dx, dy, dz);
        fx = __builtin_fmaf(fac, dx, fx);
        fy = __builtin_fmaf(fac, dy, fy);
        fz = __builtin_fmaf(fac, dz, fz);
    });
}

// The same sum, each batch of entries loaded as it is needed (see step_resident).
template <bool ACT, int EX, int BATCH>
__device__ __forceinline__ void gather_batches(uint32_t tbase, const float* __restrict__ sf, float4 xi, int s,
                                             int nslice, const int32_t* __restrict__ slice_ptr,
                                             const uint32_t* __restrict__ packed, float& fx, float& fy, float& fz) {
    fx = fy = fz = 0.0f;
    s = __builtin_amdgcn_readfirstlane(s);
    if (s >= nslice) return;
    const int lane = threadIdx.x & 63;
    const int e0 = __builtin_amdgcn_readfirstlane(slice_ptr[s]);
    const int w = __builtin_amdgcn_readfirstlane((slice_ptr[s + 1] - e0) >> 6);
    const uint32_t* pp = packed + e0 + lane;
    auto one = [&](uint32_t q) {
        uint32_t xa, ca, gi;
        decode_entry<ACT>(q, tbase, xa, ca, gi);
        const float4 xj = lds_f4(xa);
        const float4 c = lds_f4(ca);
        const float g = ACT ? sf[gi] : 1.0f;
        float dx, dy, dz;
        const float fac = hooke_fac_tab<ACT, EX>(xi, xj, c, g, dx, dy, dz);
        fx = __builtin_fmaf(fac, dx, fx);
        fy = __builtin_fmaf(fac, dy, fy);
        fz = __builtin_fmaf(fac, dz, fz);
    };
    int r = 0;
    for (; r + BATCH <= w; r += BATCH) {
        uint32_t q[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) q[u] = pp[(r + u) * 64];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) one(q[u]);
    }
    for (; r < w; ++r) one(pp[r * 64]);
}

// The same sum over 16-bit entries (passive simulations whose LDS slots and (k, L0) pairs fit
// together in 16 bits): neighbour slot << tb | pair index.  Half the entry stream of the
// 32-bit form, which is most of what a step reads from HBM.
template <int EX, int BATCH>
__device__ __forceinline__ void gather_narrow(uint32_t tbase, float4 xi, RowWalk<CompactRows<uint16_t>, BATCH>& walk,
                                              int tb, float& fx, float& fy, float& fz) {
    fx = fy = fz = 0.0f;
    const uint32_t tmask = (1u << tb) - 1u;
    walk.template run<kPart<EX, BATCH>>([&](uint32_t q) {
        const float4 xj = lds_f4((q >> tb) << 4);
        const float4 c = lds_f4(((q & tmask) << 4) | tbase);
        float dx, dy, dz;
        const float fac = hooke_fac_tab<false, EX>(xi, xj, c, 1.0f, dx, dy, dz);
        fx = __builtin_fmaf(fac, dx, fx);
        fy = __builtin_fmaf(fac, dy, fy);
        fz = __builtin_fmaf(fac, dz, fz);
    });
}

// Split form of the same sum, in two passes over the workgroup's LDS.
// Spring pass: every spring with an end among the workgroup's masses is evaluated once (a
// spring between two of them is shared; one to a halo mass is evaluated here and again by
// the workgroup that owns the other end), its force factor stored in LDS (sfac).  Record
// word: LDS slot of the first end (bits 0-9, always a workgroup mass), LDS slot of the other
// end (bits 10-22), (k, L0) pair index (bits 23-31); actuated springs carry their local
// factor index in a parallel 16-bit stream.
constexpr uint32_t kRecA = 10, kRecB = 13;

template <bool ACT, bool EXACT, int BATCH>
__device__ __forceinline__ void spring_pass(const float4* __restrict__ sx, uint32_t tbase,
                                            const float* __restrict__ sf, float* __restrict__ sfac,
                                            const uint32_t* __restrict__ rec, const uint16_t* __restrict__ rgrp,
                                            int n_sp, int block, float safe) {
    const int lane = threadIdx.x & 63;
    const int w0 = (int)(threadIdx.x & ~63u);
    if (threadIdx.x == 0) sfac[n_sp] = 0.0f;  // the factor of the padding entries
    for (int j0 = __builtin_amdgcn_readfirstlane(w0); j0 < n_sp; j0 += BATCH * block) {
        uint32_t r[BATCH];
        int gi[BATCH];
        float g[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {  // lanes past the end re-read the last record
            const int j = min(j0 + u * block + lane, n_sp - 1);
            r[u] = rec[j];
            if (ACT) gi[u] = rgrp[j];
        }
        // every load is issued before the first of them is waited for (left to itself the compiler may wait
        // for each group index in turn)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
            if (ACT) g[u] = sf[gi[u]];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int j = j0 + u * block + lane;
            const float4 xa = lds_f4((r[u] << 4) & (((1u << kRecA) - 1u) << 4));
            const float4 xb = lds_f4((r[u] >> (kRecA - 4)) & (((1u << kRecB) - 1u) << 4));
            const float4 c = lds_f4(((r[u] >> (kRecA + kRecB)) << 4) | tbase);
            bool plain = !EXACT;
            if (EXACT) {
                const float m = fminf(fminf(fabsf(xa.x), fabsf(xa.y)), fabsf(xa.z));
                plain = __builtin_amdgcn_ballot_w64(j < n_sp && !(m >= safe)) == 0;
            }
            float dx, dy, dz, fac;
            if (plain) fac = hooke_fac_tab<ACT, kPlain>(xa, xb, c, ACT ? g[u] : 1.0f, dx, dy, dz);
            else fac = hooke_fac_tab<ACT, kExactAll>(xa, xb, c, ACT ? g[u] : 1.0f, dx, dy, dz);
            if (j < n_sp) sfac[j] = fac;
        }
    }
}

// Gather pass: each lane walks its mass's entries in the usual order; an entry holds the
// neighbour's LDS slot (bits 0-12) and the index of the spring's factor in sfac (bits 13-31).
// Its arithmetic is light, so the entry loads would sit exposed: the first kPre entries of
// the slice are loaded (`prefetch_entries`) before the spring pass and consumed after it.
constexpr int kPre = 16;

struct SliceEntries {
    const uint32_t* pp;  // this lane's first entry
    int w;               // entries per lane (uniform over the wavefront)
    uint32_t pre[kPre];
};

__device__ __forceinline__ void prefetch_entries(SliceEntries& se, int s, int nslice,
                                                 const int32_t* __restrict__ slice_ptr,
                                                 const uint32_t* __restrict__ packed) {
    s = __builtin_amdgcn_readfirstlane(s);
    se.w = 0;
    se.pp = packed;
    if (s >= nslice) return;
    const int e0 = __builtin_amdgcn_readfirstlane(slice_ptr[s]);
    se.w = __builtin_amdgcn_readfirstlane((slice_ptr[s + 1] - e0) >> 6);
    se.pp = packed + e0 + (threadIdx.x & 63);
#pragma unroll
    for (int u = 0; u < kPre; ++u)
        if (u < se.w) se.pre[u] = se.pp[u * 64];
}

template <int BATCH>
__device__ __forceinline__ void gather_split(uint32_t fbase, float4 xi, const SliceEntries& se, float& fx, float& fy,
                                             float& fz) {
    fx = fy = fz = 0.0f;
    auto one = [&](uint32_t q) {
        const float4 xj = lds_f4((q & ((1u << kSlotBits) - 1u)) << 4);
        const float fac = lds_f1(((q >> kSlotBits) << 2) + fbase);
        fx = __builtin_fmaf(fac, xj.x - xi.x, fx);
        fy = __builtin_fmaf(fac, xj.y - xi.y, fy);
        fz = __builtin_fmaf(fac, xj.z - xi.z, fz);
    };
#pragma unroll
    for (int u = 0; u < kPre; ++u)
        if (u < se.w) one(se.pre[u]);
    int r = kPre;
    for (; r + BATCH <= se.w; r += BATCH) {
        uint32_t q[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) q[u] = se.pp[(r + u) * 64];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) one(q[u]);
    }
    for (; r < se.w; ++r) one(se.pp[r * 64]);
}

struct StepArgs {
    const float4* __restrict__ xin;
    const float* __restrict__ vin;
    float4* __restrict__ xout;
    float* __restrict__ vout;
    const int32_t* __restrict__ slice_ptr;
    const uint16_t* __restrict__ nbr;
    const float2* __restrict__ kl;
    const uint16_t* __restrict__ grp;
    const int32_t* __restrict__ halo_ptr;
    const int32_t* __restrict__ halo_idx;
    const uint16_t* __restrict__ lane_mass;
    const float* __restrict__ factor;
    const float* __restrict__ fext;
    float* __restrict__ vstar_out;   // optional: velocity before friction and damping (adjoint recompute)
    const uint32_t* __restrict__ packed;   // compact entries (see gather_table), or null
    const uint16_t* __restrict__ narrow;   // 16-bit compact entries (see gather_narrow), or null
    const float4* __restrict__ table;      // (k, L0, L0^2 in FP64) of the compact entries
    const int2* __restrict__ blk_groups;   // per workgroup: first factor index and count
    const uint32_t* __restrict__ sp_rec;   // split form: spring records, workgroup after workgroup
    const uint16_t* __restrict__ sp_grp;   // split form: local actuation factor index per record
    const int32_t* __restrict__ sp_ptr;    // split form: first record of each workgroup
    int n, nblk, nslice, block, n_table, lds_slots, max_local_groups;
    int narrow_tb;                         // pair-index bits of the 16-bit entries
    // fused actuation (actuated table forms): each workgroup computes its factors for step
    // n = *step_in from phase and amp; one thread stores n + 1 to *step_out (the other slot of
    // the counter pair, so no workgroup of this launch reads it)
    int fuse;
    const float* __restrict__ phase;
    const float* __restrict__ amp;
    const long long* step_in;
    long long* step_out;
    const ActuationState* act;
};

// Difference mode of a wavefront (uniform across it).  A coordinate at least `safe` away from
// zero makes its difference with any neighbour closer than safe/2 exact (Sterbenz), and a
// spring longer than that is far from rest, where a one-ulp error in d is negligible; so an
// axis needs the residual terms only if some mass of the wavefront is nearer its plane.
__device__ __forceinline__ int difference_mode(float4 xi, float safe) {
    const bool nx = __builtin_amdgcn_ballot_w64(!(fabsf(xi.x) >= safe)) != 0;
    const bool ny = __builtin_amdgcn_ballot_w64(!(fabsf(xi.y) >= safe)) != 0;
    const bool nz = __builtin_amdgcn_ballot_w64(!(fabsf(xi.z) >= safe)) != 0;
    return (nx || ny) ? kExactAll : nz ? kExactZ : kPlain;
}

// The exact-difference loop holds more live values per entry; it loads half as far ahead so
// that it does not raise the kernel's register count (and cut its occupancy).
template <int BATCH>
constexpr int kExactBatch = BATCH > 2 ? BATCH / 2 : BATCH;

// Per-launch arguments of the resident form (see step_resident).
struct ResidentArgs {
    const float* __restrict__ phase;
    const float* __restrict__ amp;
    unsigned long long cycles;
    const long long* step_in;   // step index of the input state (one slot of the counter pair)
    long long* step_out;        // receives the index after the launch (the other slot)
    int steps;
    float dtv0;
    int staged;                 // compact entries copied into LDS after the factors (0: none)
};

// Step modes: explicit (k, L0) per entry, compact entries with the parameter table, split.
enum : int { kExplicit = 0, kTable = 1, kSplit = 2, kNarrow = 3 };

// Elapsed fraction of an actuation period at step n, frac(n f dt), formed exactly in 64-bit
// fixed point (n * cycles wraps modulo 2^64), and the factor 1 + A sin(2 pi u + phi).
__device__ __forceinline__ float period_fraction(long long n, unsigned long long cycles) {
    const unsigned long long frac = (unsigned long long)n * cycles;
    return (float)(unsigned)(frac >> 32) * 0x1p-32f;
}
__device__ __forceinline__ float actuation_factor(float amp, float phase, float u) {
    return __builtin_fmaf(amp, sinf(__builtin_fmaf(6.28318531f, u, phase)), 1.0f);
}

// Body forces, contact, friction, damping and the symplectic Euler update of one mass with
// spring force f: v* = v + dtv a (v* is stored to vstar when given), Coulomb clamp, damping,
// x' = x + dt v'; a fixed mass (1/m = 0) keeps x and gets v' = 0.  dtv is dt except in
// Verlet's first step (dt / 2).
__device__ __forceinline__ void integrate(const StepParams& p, float dtv, float4 xi, float fx, float fy, float fz,
                                          const float* __restrict__ fext, float& vx, float& vy, float& vz,
                                          float4& xo, float* __restrict__ vstar) {
    const float inv_m = xi.w;
    float ax = __builtin_fmaf(fx, inv_m, p.gx);
    float ay = __builtin_fmaf(fy, inv_m, p.gy);
    float az = __builtin_fmaf(fz, inv_m, p.gz);
    if (fext) {
        ax = __builtin_fmaf(fext[0], inv_m, ax);
        ay = __builtin_fmaf(fext[1], inv_m, ay);
        az = __builtin_fmaf(fext[2], inv_m, az);
    }
    float fn = 0.0f;
    if (p.ground) {
        const float pen = p.ground_z - xi.z;
        fn = pen > 0.0f ? p.ground_k * pen : 0.0f;
        az = __builtin_fmaf(fn, inv_m, az);
    }
    vx = __builtin_fmaf(dtv, ax, vx);
    vy = __builtin_fmaf(dtv, ay, vy);
    vz = __builtin_fmaf(dtv, az, vz);
    if (vstar) {
        vstar[0] = vx;
        vstar[1] = vy;
        vstar[2] = vz;
    }
    if (fn > 0.0f) {
        // Coulomb clamp: the tangential speed loses mu F_n dtv / m, or stops
        const float c = p.ground_mu * fn * dtv * inv_m;
        const float sp = __builtin_sqrtf(vx * vx + vy * vy);
        const float sc = sp > c ? (sp - c) / sp : 0.0f;
        vx *= sc;
        vy *= sc;
    }
    vx *= p.damp;
    vy *= p.damp;
    vz *= p.damp;
    xo = make_float4(__builtin_fmaf(p.dt, vx, xi.x), __builtin_fmaf(p.dt, vy, xi.y), __builtin_fmaf(p.dt, vz, xi.z),
                     inv_m);
    if (inv_m == 0.0f) {  // fixed mass
        xo = xi;
        vx = vy = vz = 0.0f;
    }
}

// One time step of the masses of workgroup-block b: gather, body forces, contact, friction,
// damping, symplectic Euler, fixed masses.
template <bool ACT, bool EXACT, int BATCH, int MODE, bool STAGE = false>
__device__ __forceinline__ void step_block(float4* __restrict__ sx, const StepArgs& a, const StepParams& p, int b,
                                           float u) {
    constexpr bool TABLE = MODE != kExplicit;
    const int t = (int)threadIdx.x, base = b * a.block;
    const uint32_t tbase = table_base(a.lds_slots);
    float4* st = reinterpret_cast<float4*>(reinterpret_cast<char*>(sx) + tbase);
    float* sf = reinterpret_cast<float*>(st + a.n_table);
    float* sfac = sf + a.max_local_groups + 1;
    // every load that depends on nothing staged is issued before the first is waited for: the
    // lane's mass, the first halo index, positions, the first batch of entries, the table's
    // first part, then what hangs on those
    const int own = a.lane_mass[base + t];
    float4 xt = make_float4(0.f, 0.f, 0.f, 0.f), xh = xt, tab = xt;
    if (base + t < a.n) xt = a.xin[base + t];   // before the halo's, which first waits for halo_ptr
    const int h0 = a.halo_ptr[b], h1 = a.halo_ptr[b + 1];
    const int hj = h0 + t < h1 ? a.halo_idx[h0 + t] : -1;
    if (TABLE && t < a.n_table) tab = a.table[t];
    const int2 bg = TABLE && ACT ? a.blk_groups[b] : make_int2(0, 0);
    const int s = (base + t) >> 6;
    SliceEntries se;
    RowWalk<CompactRows<uint32_t>, BATCH> rt{{a.packed}};
    RowWalk<CompactRows<uint16_t>, BATCH> rn{{a.narrow}};
    if (MODE == kSplit) prefetch_entries(se, s, a.nslice, a.slice_ptr, a.packed);
    else if (MODE == kNarrow) rn.start(s, a.nslice, a.slice_ptr);   // passive only (the host never picks it for actuation)
    else if (TABLE) rt.start(s, a.nslice, a.slice_ptr);
    if (hj >= 0) xh = a.xin[hj];
    // velocities read in mass order (one contiguous run), handed to each mass's lane through LDS below
    float vt0 = 0.0f, vt1 = 0.0f, vt2 = 0.0f;
    if (STAGE && base + t < a.n) {
        const long q = 3 * (long)(base + t);
        vt0 = a.vin[q + 0];
        vt1 = a.vin[q + 1];
        vt2 = a.vin[q + 2];
    }
    if (TABLE && ACT) {
        if (a.fuse) {   // the same formula as actuation_kernel, for this workgroup's factors only
            for (int q = t; q <= bg.y; q += a.block)
                sf[q] = q ? actuation_factor(a.amp[bg.x + q - 1], a.phase[bg.x + q - 1], u) : 1.0f;
        } else {
            for (int q = t; q <= bg.y; q += a.block) sf[q] = q ? a.factor[bg.x + q - 1] : 1.0f;
        }
    }
    if (TABLE) {
        if (t < a.n_table) st[t] = tab;
        for (int q = t + a.block; q < a.n_table; q += a.block) st[q] = a.table[q];
    }
    sx[t] = xt;
    if (hj >= 0) sx[a.block + t] = xh;
    for (int h = h0 + t + a.block; h < h1; h += a.block) sx[a.block + (h - h0)] = a.xin[a.halo_idx[h]];
    const float safe = ACT ? a.act->safe : p.safe;   // here, so that no scalar load above is waited for with it
    __syncthreads();
    const float4 xi = sx[own];
    float fx, fy, fz;
    if (MODE == kSplit) {
        const int r0 = a.sp_ptr[b];
        spring_pass<ACT, EXACT, BATCH>(sx, tbase, sf, sfac, a.sp_rec + r0, ACT ? a.sp_grp + r0 : nullptr,
                                       a.sp_ptr[b + 1] - r0, a.block, safe);
        __syncthreads();
        gather_split<BATCH>(tbase + (uint32_t)(reinterpret_cast<char*>(sfac) - reinterpret_cast<char*>(st)), xi, se,
                            fx, fy, fz);
    } else {
        const int mode = EXACT ? difference_mode(xi, safe) : kPlain;
        if (MODE == kNarrow) {
            if (mode == kPlain) gather_narrow<kPlain, BATCH>(tbase, xi, rn, a.narrow_tb, fx, fy, fz);
            else if (mode == kExactZ) gather_narrow<kExactZ, BATCH>(tbase, xi, rn, a.narrow_tb, fx, fy, fz);
            else gather_narrow<kExactAll, BATCH>(tbase, xi, rn, a.narrow_tb, fx, fy, fz);
        } else if (TABLE) {
            if (mode == kPlain) gather_table<ACT, kPlain, BATCH>(tbase, sf, xi, rt, fx, fy, fz);
            else if (mode == kExactZ) gather_table<ACT, kExactZ, BATCH>(tbase, sf, xi, rt, fx, fy, fz);
            else gather_table<ACT, kExactAll, BATCH>(tbase, sf, xi, rt, fx, fy, fz);
        } else {
            if (mode == kPlain) gather<ACT, kPlain, BATCH>(sx, xi, s, a.nslice, a.slice_ptr, a.nbr, a.kl, a.grp, a.factor, fx, fy, fz);
            else if (mode == kExactZ)
                gather<ACT, kExactZ, BATCH>(sx, xi, s, a.nslice, a.slice_ptr, a.nbr, a.kl, a.grp, a.factor, fx, fy, fz);
            else gather<ACT, kExactAll, kExactBatch<BATCH>>(sx, xi, s, a.nslice, a.slice_ptr, a.nbr, a.kl, a.grp, a.factor, fx, fy, fz);
        }
    }
    const int i = base + own;
    if (!STAGE) {
        if (i >= a.n) return;
        float vx = a.vin[3 * i + 0], vy = a.vin[3 * i + 1], vz = a.vin[3 * i + 2];
        float4 xo;
        integrate(p, p.dtv, xi, fx, fy, fz, a.fext ? a.fext + 3 * i : nullptr, vx, vy, vz, xo,
                  a.vstar_out ? a.vstar_out + 3 * i : nullptr);
        a.xout[i] = xo;
        a.vout[3 * i + 0] = vx;
        a.vout[3 * i + 1] = vy;
        a.vout[3 * i + 2] = vz;
        return;
    }
    // The lane->mass map scatters a wavefront's masses over the block, and scattered 16- and
    // 12-byte accesses reach HBM as partly used lines: velocities come in (loaded above in
    // mass order) and the new state goes out through LDS (the staged positions and tables
    // are no longer read), one contiguous run per array.  The launch provides 40 bytes of LDS
    // per mass for it.  Two more barriers: a memory-bound system gains (the actuated
    // population: 317 -> 298 us per step), a compute-bound one loses (the 16-bit-entry
    // cantilever: 18.5 -> 20.6 us), so only the actuated 32-bit table form has the staged
    // variant, taken where the step's bytes exceed the Infinity Cache.
    __syncthreads();
    float4* ox = sx;
    float* ov = reinterpret_cast<float*>(sx + a.block);
    float* ovin = ov + 3 * a.block;
    ovin[3 * threadIdx.x + 0] = vt0;
    ovin[3 * threadIdx.x + 1] = vt1;
    ovin[3 * threadIdx.x + 2] = vt2;
    __syncthreads();
    float vx = 0.0f, vy = 0.0f, vz = 0.0f;
    float4 xo;
    if (i < a.n) {
        vx = ovin[3 * own + 0];
        vy = ovin[3 * own + 1];
        vz = ovin[3 * own + 2];
        integrate(p, p.dtv, xi, fx, fy, fz, a.fext ? a.fext + 3 * i : nullptr, vx, vy, vz, xo,
                  a.vstar_out ? a.vstar_out + 3 * i : nullptr);
    }
    if (i < a.n) {
        ox[own] = xo;
        ov[3 * own + 0] = vx;
        ov[3 * own + 1] = vy;
        ov[3 * own + 2] = vz;
    }
    __syncthreads();
    const int cnt = min(a.block, a.n - base);
    for (int q = threadIdx.x; q < cnt; q += a.block) a.xout[base + q] = ox[q];
    for (int q = threadIdx.x; q < 3 * cnt; q += a.block) a.vout[3 * (long)base + q] = ov[q];
}

// A fused-actuation launch hands the next one its step index through the other slot of the
// counter pair (the next launch reads that slot; the kernel boundary orders the two).  Returns
// this step's fraction of an actuation period.
__device__ __forceinline__ float advance_step(const StepArgs& a) {
    const long long n_step = *a.step_in;
    const unsigned long long cycles = a.act->cycles;   // both reads before the store: scalar loads
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.step_out = n_step + 1;
    return period_fraction(n_step, cycles);
}

template <bool ACT, bool EXACT, int BATCH, int MODE, bool STAGE = false>
__global__ void __launch_bounds__(1024) step_kernel(StepArgs a, StepParams p) {
    extern __shared__ float4 sx[];
    constexpr bool FUSABLE = ACT && MODE != kExplicit;
    const int b = logical_block(a.nblk);
    const float u = FUSABLE && a.fuse ? advance_step(a) : 0.0f;
    if (b < a.nblk) step_block<ACT, EXACT, BATCH, MODE, STAGE>(sx, a, p, b, u);
}

// Several lanes per mass (LPM = 2 or 4; compact table forms): lane j of a mass's group walks its
// incidence rows j, j + LPM, ... and the groups' partial sums are combined by a fixed pairing
// of cross-lane exchanges (the same value in every lane of the group).  More wavefronts for
// the same masses, each with a shorter dependent chain: for bodies too small to fill the chip.
// The sum is grouped differently from the one-lane form, so the two agree to rounding only.
//
// Such a step is a chain of latencies (the 12.7k-mass quadruped: under one wavefront per SIMD,
// 3% of the VALU's issue slots), so each lane loads its entries before the workgroup's barrier,
// beside the halo's index -> position chain, and reads all its neighbours from LDS before the
// first spring's arithmetic: 5.4 -> 4.8 us per step (two rows at a time after the barrier: a
// memory, an LDS and an arithmetic latency for each pair).  EARLY: chosen by lanes_early.
constexpr int kLaneGroup = 8;   // rows whose LDS reads are in flight together
// rows of a lane held in registers: all of a voxel node's 26 (4 lanes: 7, 2 lanes: 13)
template <int LPM>
constexpr int kLanePre = LPM == 2 ? 2 * kLaneGroup : kLaneGroup;
typedef uint32_t lane_rows_vec __attribute__((ext_vector_type(2 * kLaneGroup)));   // a vector, never an array in memory

template <int LPM, bool NARROW>
struct LaneRows {
    const uint32_t* __restrict__ packed;
    const uint16_t* __restrict__ narrow;
    int e;       // this lane's entry of incidence row 0 (row r: 64 r further)
    int w;       // incidence rows of the slice
    int count;   // rows per lane, counting a last one that some lanes of a group may lack
    lane_rows_vec q;

    // the lane's k-th entry; a lane without one gets an entry of its own mass (used with factor 0)
    __device__ __forceinline__ uint32_t row(int k, int sub, bool& ok) const {
        ok = k * LPM + sub < w;
        const int r = ok ? k * LPM + sub : k > 0 ? (k - 1) * LPM + sub : 0;
        return NARROW ? (uint32_t)narrow[e + r * 64] : packed[e + r * 64];
    }
    template <bool EARLY>
    __device__ __forceinline__ void load(int s, int lane, int sub, int nslice, const int32_t* __restrict__ slice_ptr) {
        s = __builtin_amdgcn_readfirstlane(s);
        e = w = count = 0;
        if (s >= nslice) return;
        const int e0 = __builtin_amdgcn_readfirstlane(slice_ptr[s]);
        w = __builtin_amdgcn_readfirstlane((slice_ptr[s + 1] - e0) >> 6);
        e = e0 + lane;
        count = (w + LPM - 1) / LPM;
        if (!EARLY || count == 0) return;
        bool ok;
#pragma unroll
        for (int u = 0; u < kLanePre<LPM>; ++u) q[u] = row(min(u, count - 1), sub, ok);   // stays inside the slice
    }
};

// N rows of the lane from their entries q[BASE ...]: every LDS read first, then the springs in row
// order.  Only the slice's last row can be missing in some lanes (ok_last).
template <bool ACT, int EX, bool NARROW, int BASE, int N>
__device__ __forceinline__ void lane_springs(uint32_t tbase, const float* __restrict__ sf, float4 xi, int tb,
                                             const lane_rows_vec& q, bool ok_last, float& fx, float& fy, float& fz) {
    const uint32_t tmask = (1u << tb) - 1u;
    lds_vec4 xj[N], c[N];
    float g[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        uint32_t xa, ca, gi = 0;
        if (NARROW) {
            xa = (q[BASE + u] >> tb) << 4;
            ca = ((q[BASE + u] & tmask) << 4) | tbase;
        } else {
            decode_entry<ACT>(q[BASE + u], tbase, xa, ca, gi);
        }
        xj[u] = lds_v4(xa);
        c[u] = lds_v4(ca);
        g[u] = ACT ? sf[gi] : 1.0f;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        float dx, dy, dz;
        float fac = hooke_fac_tab<ACT, EX>(xi, make_float4(xj[u].x, xj[u].y, xj[u].z, xj[u].w),
                                           make_float4(c[u].x, c[u].y, c[u].z, c[u].w), g[u], dx, dy, dz);
        if (u == N - 1) fac = ok_last ? fac : 0.0f;
        fx = __builtin_fmaf(fac, dx, fx);
        fy = __builtin_fmaf(fac, dy, fy);
        fz = __builtin_fmaf(fac, dz, fz);
    }
}

// The first `count` (at most kLaneGroup) rows of q[BASE ...]; count is uniform over the wavefront.
template <bool ACT, int EX, bool NARROW, int BASE>
__device__ __forceinline__ void lane_group(int count, uint32_t tbase, const float* __restrict__ sf, float4 xi, int tb,
                                           const lane_rows_vec& q, bool ok_last, float& fx, float& fy, float& fz) {
    switch (count) {
#define CRONOS_ROWS(N) \
    case N: lane_springs<ACT, EX, NARROW, BASE, N>(tbase, sf, xi, tb, q, ok_last, fx, fy, fz); break;
        CRONOS_ROWS(1)
        CRONOS_ROWS(2)
        CRONOS_ROWS(3)
        CRONOS_ROWS(4)
        CRONOS_ROWS(5)
        CRONOS_ROWS(6)
        CRONOS_ROWS(7)
        CRONOS_ROWS(8)
#undef CRONOS_ROWS
        default: break;
    }
}

// A lane's rows two at a time, each pair loaded when it is needed.
template <bool ACT, int EX, int LPM, bool NARROW>
__device__ __forceinline__ void lane_pairs(uint32_t tbase, const float* __restrict__ sf, float4 xi, int sub, int tb,
                                           const LaneRows<LPM, NARROW>& rows, float& fx, float& fy, float& fz) {
    const uint32_t tmask = (1u << tb) - 1u;
    auto one = [&](uint32_t q) {
        uint32_t xa, ca, gi = 0;
        if (NARROW) {
            xa = (q >> tb) << 4;
            ca = ((q & tmask) << 4) | tbase;
        } else {
            decode_entry<ACT>(q, tbase, xa, ca, gi);
        }
        const float4 xj = lds_f4(xa);
        const float4 c = lds_f4(ca);
        const float g = ACT ? sf[gi] : 1.0f;
        float dx, dy, dz;
        const float fac = hooke_fac_tab<ACT, EX>(xi, xj, c, g, dx, dy, dz);
        fx = __builtin_fmaf(fac, dx, fx);
        fy = __builtin_fmaf(fac, dy, fy);
        fz = __builtin_fmaf(fac, dz, fz);
    };
    constexpr int B = 2;
    for (int k = 0; k < rows.count; k += B) {
        uint32_t q[B];
        bool ok[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int r = (k + u) * LPM + sub, e = rows.e + r * 64;
            ok[u] = r < rows.w;
            q[u] = ok[u] ? (NARROW ? (uint32_t)rows.narrow[e] : rows.packed[e]) : 0u;
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (ok[u]) one(q[u]);
    }
}

template <bool ACT, int EX, int LPM, bool NARROW>
__device__ __forceinline__ void lane_early(uint32_t tbase, const float* __restrict__ sf, float4 xi, int sub, int tb,
                                           const LaneRows<LPM, NARROW>& rows, float& fx, float& fy, float& fz) {
    const bool ok_last = (rows.count - 1) * LPM + sub < rows.w;
    auto ok = [&](int end) { return end < rows.count || ok_last; };   // of a group that ends before row `end`
    const int n0 = min(rows.count, kLaneGroup);
    lane_group<ACT, EX, NARROW, 0>(n0, tbase, sf, xi, tb, rows.q, ok(n0), fx, fy, fz);
    if (kLanePre<LPM> > kLaneGroup && rows.count > kLaneGroup) {
        const int n1 = min(rows.count - kLaneGroup, kLaneGroup);
        lane_group<ACT, EX, NARROW, kLanePre<LPM> - kLaneGroup>(n1, tbase, sf, xi, tb, rows.q, ok(kLaneGroup + n1), fx, fy,
                                                               fz);
    }
    for (int k = kLanePre<LPM>; k < rows.count; k += 4) {   // bodies of higher degree
        lane_rows_vec q;
        bool have;
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = rows.row(min(k + u, rows.count - 1), sub, have);
        const int n = min(rows.count - k, 4);
        lane_group<ACT, EX, NARROW, 0>(n, tbase, sf, xi, tb, q, ok(k + n), fx, fy, fz);
    }
}

template <bool ACT, int EX, int LPM, bool NARROW, bool EARLY>
__device__ __forceinline__ void gather_lanes(uint32_t tbase, const float* __restrict__ sf, float4 xi, int sub, int tb,
                                             const LaneRows<LPM, NARROW>& rows, float& fx, float& fy, float& fz) {
    fx = fy = fz = 0.0f;
    if (EARLY) lane_early<ACT, EX, LPM, NARROW>(tbase, sf, xi, sub, tb, rows, fx, fy, fz);
    else lane_pairs<ACT, EX, LPM, NARROW>(tbase, sf, xi, sub, tb, rows, fx, fy, fz);
#pragma unroll
    for (int o = 1; o < LPM; o <<= 1) {
        fx += __shfl_xor(fx, o, 64);
        fy += __shfl_xor(fy, o, 64);
        fz += __shfl_xor(fz, o, 64);
    }
}

// One step with LPM lanes per mass: a workgroup of block * LPM threads stages its block's
// positions and halo, thread t serves mass lane t / LPM; the first lane of each mass
// integrates.  Compact table forms (32- or 16-bit entries), one workgroup per block.
template <bool ACT, bool EXACT, int LPM, bool NARROW, bool EARLY>
__global__ void __launch_bounds__(1024) step_lanes_kernel(StepArgs a, StepParams p) {
    extern __shared__ float4 sx[];
    // the arguments that the first loads need, fetched together (one scalar-cache latency, not
    // one for each use)
    asm volatile("" ::"s"(a.xin), "s"(a.vin), "s"(a.slice_ptr), "s"(a.halo_ptr), "s"(a.halo_idx), "s"(a.lane_mass),
                 "s"(NARROW ? (const void*)a.narrow : (const void*)a.packed), "s"(a.table), "s"(a.n), "s"(a.nblk),
                 "s"(a.nslice), "s"(a.block), "s"(a.n_table), "s"(a.lds_slots));
    const int b = logical_block(a.nblk);
    const float safe = ACT ? a.act->safe : p.safe;
    const float u = ACT && a.fuse ? advance_step(a) : 0.0f;
    if (b >= a.nblk) return;
    const int t = (int)threadIdx.x, nt = (int)blockDim.x;
    const int m = t / LPM, sub = t % LPM;
    const int base = b * a.block;
    // every load that depends on nothing staged is issued here: the first halo index, this
    // lane's mass, its own position, its entries, then what hangs on those
    const int h0 = a.halo_ptr[b], h1 = a.halo_ptr[b + 1];
    const int own = a.lane_mass[base + m];
    const int hj = h0 + t < h1 ? a.halo_idx[h0 + t] : -1;
    float4 xt = make_float4(0.f, 0.f, 0.f, 0.f), xh = xt;
    if (t < a.block && base + t < a.n) xt = a.xin[base + t];
    LaneRows<LPM, NARROW> rows;
    rows.packed = a.packed;
    rows.narrow = a.narrow;
    rows.template load<EARLY>((base + m) >> 6, m & 63, sub, a.nslice, a.slice_ptr);
    const uint32_t tbase = table_base(a.lds_slots);
    float4* st = reinterpret_cast<float4*>(reinterpret_cast<char*>(sx) + tbase);
    float* sf = reinterpret_cast<float*>(st + a.n_table);
    if (hj >= 0) xh = a.xin[hj];
    const int i = base + own;
    const bool mine = sub == 0 && i < a.n;
    float vx = 0.0f, vy = 0.0f, vz = 0.0f;
    if (mine) {
        vx = a.vin[3 * i + 0];
        vy = a.vin[3 * i + 1];
        vz = a.vin[3 * i + 2];
    }
    for (int q = t; q < a.n_table; q += nt) st[q] = a.table[q];
    if (ACT) {
        const int2 bg = a.blk_groups[b];
        if (a.fuse) {
            for (int q = t; q <= bg.y; q += nt)
                sf[q] = q ? actuation_factor(a.amp[bg.x + q - 1], a.phase[bg.x + q - 1], u) : 1.0f;
        } else {
            for (int q = t; q <= bg.y; q += nt) sf[q] = q ? a.factor[bg.x + q - 1] : 1.0f;
        }
    }
    if (t < a.block) sx[t] = xt;   // block * LPM threads: one round
    if (hj >= 0) sx[a.block + t] = xh;
    for (int h = h0 + t + nt; h < h1; h += nt) sx[a.block + (h - h0)] = a.xin[a.halo_idx[h]];
    __syncthreads();
    const float4 xi = sx[own];
    float fx, fy, fz;
    const int mode = EXACT ? difference_mode(xi, safe) : kPlain;
    if (mode == kPlain)
        gather_lanes<ACT, kPlain, LPM, NARROW, EARLY>(tbase, sf, xi, sub, a.narrow_tb, rows, fx, fy, fz);
    else if (mode == kExactZ)
        gather_lanes<ACT, kExactZ, LPM, NARROW, EARLY>(tbase, sf, xi, sub, a.narrow_tb, rows, fx, fy, fz);
    else
        gather_lanes<ACT, kExactAll, LPM, NARROW, EARLY>(tbase, sf, xi, sub, a.narrow_tb, rows, fx, fy, fz);
    if (!mine) return;
    float4 xo;
    integrate(p, p.dtv, xi, fx, fy, fz, a.fext ? a.fext + 3 * i : nullptr, vx, vy, vz, xo,
              a.vstar_out ? a.vstar_out + 3 * i : nullptr);
    a.xout[i] = xo;
    a.vout[3 * i + 0] = vx;
    a.vout[3 * i + 1] = vy;
    a.vout[3 * i + 2] = vz;
}

// One step by explicit entries with four lanes per mass, bitwise the one-lane form's: lane j of a mass
// evaluates rows j, j + 4, ..., and every lane adds the four lanes' forces in row order (their
// factors and differences broadcast within the quad by register moves).  The sums cost each lane
// what they cost one, but they are 3 of some 40 operations a row: on bodies of under one wavefront per
// SIMD, where a wavefront issues alone, the rest goes four times as fast.
// A workgroup is one slice of 64 masses (the host's rule), and each of its four wavefronts chooses the
// difference for the slice, from all 64 positions, as the one lane-per-mass wavefront does: chosen for
// its own 16 masses, springs of many rest lengths' stretch got other bits beside a plane.
template <int Q>
__device__ __forceinline__ float quad_lane(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), Q * 0x55, 0xF, 0xF, true));
}

constexpr int kQuadPre = 7;   // rows a lane loads up front: 28 of a mass

template <bool ACT, int EX, int N>
__device__ __forceinline__ void quad_rows(const float4* __restrict__ sx, float4 xi, int slot, float2 c, float f, float& fx,
                                          float& fy, float& fz) {
    const float4 xj = sx[slot];
    float dx, dy, dz;
    const float fac = hooke_fac<EX>(xi.x, xi.y, xi.z, xj.x, xj.y, xj.z, c.x, ACT ? c.y * f : c.y, dx, dy, dz);
    auto add = [&](float g, float x, float y, float z) {
        fx = __builtin_fmaf(g, x, fx);
        fy = __builtin_fmaf(g, y, fy);
        fz = __builtin_fmaf(g, z, fz);
    };
    add(quad_lane<0>(fac), quad_lane<0>(dx), quad_lane<0>(dy), quad_lane<0>(dz));
    if (N > 1) add(quad_lane<1>(fac), quad_lane<1>(dx), quad_lane<1>(dy), quad_lane<1>(dz));
    if (N > 2) add(quad_lane<2>(fac), quad_lane<2>(dx), quad_lane<2>(dy), quad_lane<2>(dz));
    if (N > 3) add(quad_lane<3>(fac), quad_lane<3>(dx), quad_lane<3>(dy), quad_lane<3>(dz));
}

template <bool ACT, bool EXACT>
__global__ void __launch_bounds__(256) step_quads_kernel(StepArgs a, StepParams p) {
    extern __shared__ float4 sx[];
    const int b = logical_block(a.nblk);
    const float safe = ACT ? a.act->safe : p.safe;
    if (b >= a.nblk) return;
    const int t = (int)threadIdx.x, nt = (int)blockDim.x;
    const int m = t >> 2, sub = t & 3, base = b * a.block;
    const int h0 = a.halo_ptr[b], h1 = a.halo_ptr[b + 1];
    const int own = a.lane_mass[base + m];
    const int hj = h0 + t < h1 ? a.halo_idx[h0 + t] : -1;
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 xt = a.xin[min(base + min(t, a.block - 1), a.n - 1)], xh = z;
    const int s = __builtin_amdgcn_readfirstlane((base + m) >> 6);
    int e0 = 0, w = 0;
    if (s < a.nslice) {
        e0 = __builtin_amdgcn_readfirstlane(a.slice_ptr[s]);
        w = __builtin_amdgcn_readfirstlane((a.slice_ptr[s + 1] - e0) >> 6);
    }
    int slot[kQuadPre], g[kQuadPre];
    float2 c[kQuadPre];
    auto load = [&](int u, int r) {   // past the end: the last row again (an empty slice: the arrays' padding)
        const int e = e0 + (m & 63) + max(min(r + sub, w - 1), 0) * 64;
        slot[u] = a.nbr[e];
        c[u] = a.kl[e];
        if (ACT) g[u] = a.grp[e];
    };
#pragma unroll
    for (int u = 0; u < kQuadPre; ++u) load(u, 4 * u);
    if (hj >= 0) xh = a.xin[hj];
    const int i = base + own;
    const bool mine = sub == 0 && i < a.n;
    float vx = 0.0f, vy = 0.0f, vz = 0.0f;
    if (mine) {
        vx = a.vin[3 * i + 0];
        vy = a.vin[3 * i + 1];
        vz = a.vin[3 * i + 2];
    }
    if (base + t >= a.n) xt = z;
    if (t < a.block) sx[t] = xt;   // block * 4 threads: one round
    if (hj >= 0) sx[a.block + t] = xh;
    for (int h = h0 + t + nt; h < h1; h += nt) sx[a.block + (h - h0)] = a.xin[a.halo_idx[h]];
    __syncthreads();
    const float4 xi = sx[own];
    const int mode = EXACT ? difference_mode(sx[t & 63], safe) : kPlain;
    float fx = 0.0f, fy = 0.0f, fz = 0.0f;
    auto rows = [&](auto ex, int u, int left) {   // left: rows from this lane group's first on, uniform
        constexpr int EX = decltype(ex)::value;
        const float f = ACT ? a.factor[g[u]] : 1.0f;
        switch (min(left, 4)) {
        case 1: quad_rows<ACT, EX, 1>(sx, xi, slot[u], c[u], f, fx, fy, fz); break;
        case 2: quad_rows<ACT, EX, 2>(sx, xi, slot[u], c[u], f, fx, fy, fz); break;
        case 3: quad_rows<ACT, EX, 3>(sx, xi, slot[u], c[u], f, fx, fy, fz); break;
        case 4: quad_rows<ACT, EX, 4>(sx, xi, slot[u], c[u], f, fx, fy, fz); break;
        }
    };
    auto walk = [&](auto ex) {
#pragma unroll
        for (int u = 0; u < kQuadPre; ++u)
            if (4 * u < w) rows(ex, u, w - 4 * u);
        for (int r = 4 * kQuadPre; r < w; r += 4) {
            load(0, r);
            rows(ex, 0, w - r);
        }
    };
    if (mode == kPlain) walk(std::integral_constant<int, kPlain>{});
    else if (mode == kExactZ) walk(std::integral_constant<int, kExactZ>{});
    else walk(std::integral_constant<int, kExactAll>{});
    if (!mine) return;
    float4 xo;
    integrate(p, p.dtv, xi, fx, fy, fz, a.fext ? a.fext + 3 * i : nullptr, vx, vy, vz, xo,
              a.vstar_out ? a.vstar_out + 3 * i : nullptr);
    a.xout[i] = xo;
    a.vout[3 * i + 0] = vx;
    a.vout[3 * i + 1] = vy;
    a.vout[3 * i + 2] = vz;
}

// Persistent form: a fixed grid (a multiple of 8 workgroups) walks the blocks; workgroup w runs
// on XCD w % 8 and takes that XCD's contiguous eighth of the blocks in strides.
template <bool ACT, bool EXACT, int BATCH, int MODE, bool STAGE = false>
__global__ void __launch_bounds__(1024) step_persistent(StepArgs a, StepParams p) {
    extern __shared__ float4 sx[];
    const int per = (a.nblk + 7) >> 3;
    const int xcd = (int)(blockIdx.x & 7u);
    const int stride = (int)(gridDim.x >> 3);
    constexpr bool FUSABLE = ACT && MODE != kExplicit;
    const float u = FUSABLE && a.fuse ? advance_step(a) : 0.0f;
    for (int j = (int)(blockIdx.x >> 3); j < per; j += stride) {
        const int b = xcd * per + j;
        if (b >= a.nblk) break;
        step_block<ACT, EXACT, BATCH, MODE, STAGE>(sx, a, p, b, u);
        __syncthreads();  // LDS is restaged for the next block
    }
}

// Resident form for a system that fits one workgroup (at most 1024 masses, one block, the
// compact table form): K steps in one launch.  Positions stay in LDS, velocities in
// registers; each step computes its actuation factors in place (the same formula as
// actuation_kernel), gathers, integrates, and after a barrier overwrites the positions.  The
// device step counter advances by K.  The first step kicks for dtv0 (Verlet's dt / 2).
// STAGED: the compact entries are copied into LDS once (r.staged of them, after the factors),
// so no step waits on a memory load.
// AHEAD: entries are loaded a batch ahead (RowWalk), which suits workgroups of more than 512 threads: 1,000
// masses 4.40 -> 4.27 us a step.  With two wavefronts per SIMD or fewer the step is one chain, in which
// the loop by batches lets the compiler issue a batch's LDS reads together: 125 masses 2.24 us a
// step, 2.67 loaded ahead; 216 masses 2.27 / 2.62; 512 masses 2.69 / 2.71.
template <bool ACT, bool EXACT, int BATCH, bool STAGED, bool AHEAD>
__global__ void __launch_bounds__(1024) step_resident(StepArgs a, StepParams p, ResidentArgs r) {
    extern __shared__ float4 sx[];
    const uint32_t tbase = table_base(a.lds_slots);
    float4* st = reinterpret_cast<float4*>(reinterpret_cast<char*>(sx) + tbase);
    float* sf = reinterpret_cast<float*>(st + a.n_table);
    const int t = (int)threadIdx.x;
    for (int q = t; q < a.n_table; q += a.block) st[q] = a.table[q];
    RowWalk<ResidentRows, BATCH> first{{a.packed, 0}};
    if (AHEAD) first.start(t >> 6, a.nslice, a.slice_ptr);
    const uint32_t* pk = a.packed;
    if (STAGED) {
        uint32_t* se = reinterpret_cast<uint32_t*>(sf + a.max_local_groups + 1);
        for (int q = t; q < r.staged; q += a.block) se[q] = a.packed[q];
        first.rows.words = se + (first.rows.words - a.packed);
        pk = se;
    }
    sx[t] = t < a.n ? a.xin[t] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int own = a.lane_mass[t];
    const bool live = own < a.n;
    float vx = 0.f, vy = 0.f, vz = 0.f;
    if (live) {
        vx = a.vin[3 * own + 0];
        vy = a.vin[3 * own + 1];
        vz = a.vin[3 * own + 2];
    }
    const long long n0 = *r.step_in;
    const int2 bg = ACT ? a.blk_groups[0] : make_int2(0, 0);
    const float* fext = a.fext && live ? a.fext + 3 * own : nullptr;
    float4 xo = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < r.steps; ++k) {
        if (ACT) {
            const float u = period_fraction(n0 + k, r.cycles);
            for (int q = t; q <= bg.y; q += a.block)
                sf[q] = q ? actuation_factor(r.amp[bg.x + q - 1], r.phase[bg.x + q - 1], u) : 1.0f;
        }
        __syncthreads();  // positions of step k and its factors are in LDS
        const float4 xi = sx[own];
        float fx, fy, fz;
        const int mode = EXACT ? difference_mode(xi, p.safe) : kPlain;
        if (AHEAD) {
            auto walk = first;
            if (mode == kPlain) gather_table<ACT, kPlain, BATCH>(tbase, sf, xi, walk, fx, fy, fz);
            else if (mode == kExactZ) gather_table<ACT, kExactZ, BATCH>(tbase, sf, xi, walk, fx, fy, fz);
            else gather_table<ACT, kExactAll, BATCH>(tbase, sf, xi, walk, fx, fy, fz);
        } else {
            if (mode == kPlain) gather_batches<ACT, kPlain, BATCH>(tbase, sf, xi, t >> 6, a.nslice, a.slice_ptr, pk, fx, fy, fz);
            else if (mode == kExactZ)
                gather_batches<ACT, kExactZ, BATCH>(tbase, sf, xi, t >> 6, a.nslice, a.slice_ptr, pk, fx, fy, fz);
            else
                gather_batches<ACT, kExactAll, kExactBatch<BATCH>>(tbase, sf, xi, t >> 6, a.nslice, a.slice_ptr, pk, fx, fy, fz);
        }
        integrate(p, k == 0 ? r.dtv0 : p.dtv, xi, fx, fy, fz, fext, vx, vy, vz, xo, nullptr);
        __syncthreads();  // every lane has read step k's positions
        if (live) sx[own] = xo;
    }
    if (live) {
        a.xout[own] = xo;
        a.vout[3 * own + 0] = vx;
        a.vout[3 * own + 1] = vy;
        a.vout[3 * own + 2] = vz;
    }
    if (t == 0) *r.step_out = n0 + r.steps;
}

// Total force of eq. (2) + contact normal at the current state (same gather as the step).
template <bool ACT>
__global__ void __launch_bounds__(1024)
forces_kernel(const float4* __restrict__ xin, const float* __restrict__ mass, const int32_t* __restrict__ slice_ptr,
              const uint16_t* __restrict__ nbr, const float2* __restrict__ kl, const uint16_t* __restrict__ grp,
              const int32_t* __restrict__ halo_ptr, const int32_t* __restrict__ halo_idx,
              const uint16_t* __restrict__ lane_mass, const float* __restrict__ factor,
              const float* __restrict__ fext, float* __restrict__ fout, int n, int nblk, int nslice, int block,
              StepParams p) {
    extern __shared__ float4 sx[];
    const int b = logical_block(nblk);
    if (b >= nblk) return;
    const int base = b * block;
    const int own = stage_positions(sx, xin, halo_ptr, halo_idx, lane_mass, b, base, n, block);
    const float4 xi = sx[own];
    float fx, fy, fz;
    // the choice of difference of the steps that run one lane per mass (and of the explicit ones that run four), so
    // this is the force such a step integrates; several lanes per mass choose for 32 or 16 masses at a time, which
    // tells for springs of more than twice their rest length beside a coordinate plane only
    const int mode = p.exact ? difference_mode(xi, p.safe) : kPlain;
    const int s = (base + (int)threadIdx.x) >> 6;
    if (mode == kPlain) gather<ACT, kPlain, 4>(sx, xi, s, nslice, slice_ptr, nbr, kl, grp, factor, fx, fy, fz);
    else if (mode == kExactZ) gather<ACT, kExactZ, 4>(sx, xi, s, nslice, slice_ptr, nbr, kl, grp, factor, fx, fy, fz);
    else gather<ACT, kExactAll, 4>(sx, xi, s, nslice, slice_ptr, nbr, kl, grp, factor, fx, fy, fz);
    const int i = base + own;
    if (i >= n) return;
    const float m = mass[i];
    fx = __builtin_fmaf(m, p.gx, fx);
    fy = __builtin_fmaf(m, p.gy, fy);
    fz = __builtin_fmaf(m, p.gz, fz);
    if (fext) {
        fx += fext[3 * i + 0];
        fy += fext[3 * i + 1];
        fz += fext[3 * i + 2];
    }
    if (p.ground) {
        const float pen = p.ground_z - xi.z;
        if (pen > 0.0f) fz += p.ground_k * pen;
    }
    fout[3 * i + 0] = fx;
    fout[3 * i + 1] = fy;
    fout[3 * i + 2] = fz;
}

// Actuation factors 1 + A_g sin(2 pi f t_n + phi_g) of eq. (2)'s rest lengths at step n, one per
// (body, group), FP32.  The elapsed fraction of a period, frac(n f dt), is formed exactly in
// 64-bit fixed point (n * cycles wraps modulo 2^64), so the phase stays accurate to ~1e-7 rad
// however many steps have been taken.  The step index is n_explicit, or (n_explicit < 0) the
// device counter *step_in; with `advance`, one thread stores n + 1 to *step_out, the other
// slot of the counter pair, which the next launch reads.
__global__ void __launch_bounds__(256)
actuation_kernel(const float* __restrict__ phase, const float* __restrict__ amp, const ActuationState* __restrict__ act,
                 const long long* step_in, long long* step_out, float* __restrict__ factor, int n_factor, int advance,
                 long long n_explicit) {
    const long long n = n_explicit >= 0 ? n_explicit : *step_in;
    const float u = period_fraction(n, act->cycles);
    const int g = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (g < n_factor) factor[g] = actuation_factor(amp[g], phase[g], u);
    else if (g == n_factor) factor[g] = 1.0f;
    if (advance && blockIdx.x == 0 && threadIdx.x == 0) *step_out = n + 1;
}

// The factors of steps n0, n0 + 1, ..., n0 + gridDim.y - 1 (one per blockIdx.y), row k at
// out + k * stride: the same formula as actuation_kernel, for a recomputed segment at once.
__global__ void __launch_bounds__(256)
actuation_steps_kernel(const float* __restrict__ phase, const float* __restrict__ amp, unsigned long long cycles,
                       long long n0, float* __restrict__ out, int n_factor, long long stride) {
    const int k = (int)blockIdx.y;
    const float u = period_fraction(n0 + k, cycles);
    const int g = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    float* f = out + (size_t)k * (size_t)stride;
    if (g < n_factor) f[g] = actuation_factor(amp[g], phase[g], u);
    else if (g == n_factor) f[g] = 1.0f;
}

// ---------------------------------------------------------------- FP64 diagnostics

// The value of another lane of the same sixteen, by data-parallel primitive CTRL.
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// op over the wavefront's lanes, the same value in each: within sixteen lanes by data-parallel
// primitives (register moves), across them by two shuffles, which go through the LDS unit.
template <class Op>
__device__ __forceinline__ double wave_reduce(double v, Op op) {
    v = op(v, dpp_double<0xB1>(v));    // lane ^ 1
    v = op(v, dpp_double<0x4E>(v));    // lane ^ 2
    v = op(v, dpp_double<0x141>(v));   // the other half of eight
    v = op(v, dpp_double<0x140>(v));   // the other half of sixteen
    v = op(v, __shfl_xor(v, 16, 64));
    return op(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ double wave_sum(double v) {
    return wave_reduce(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_min(double v) {
    return wave_reduce(v, [](double a, double b) { return fmin(a, b); });
}
__device__ __forceinline__ double wave_max(double v) {
    return wave_reduce(v, [](double a, double b) { return fmax(a, b); });
}

// One workgroup per chunk = (workgroup-block b, masses [m0, m1) of one body).  Every term is
// widened to FP64, reduced across the wavefront with cross-lane shuffles, then across the
// workgroup's wavefronts in a fixed order.  Spring energy is counted at the lower endpoint; which
// end that is comes with the staged positions (device index in place of 1/m), and entries are loaded
// four rows at a time, the first before the staging.  A call for 640,000 masses, host included: 542 -> 70 us
// (with diag_body_kernel below); the quadruped 100 -> 31.
template <bool ACT>
__global__ void __launch_bounds__(1024)
diag_chunk_kernel(const float4* __restrict__ xin, const float* __restrict__ vin, const float* __restrict__ mass,
                  const int32_t* __restrict__ slice_ptr, const uint16_t* __restrict__ nbr,
                  const float2* __restrict__ kl, const uint16_t* __restrict__ grp,
                  const int32_t* __restrict__ halo_ptr, const int32_t* __restrict__ halo_idx,
                  const uint16_t* __restrict__ lane_mass, const float* __restrict__ factor,
                  const int4* __restrict__ chunks, double* __restrict__ part, int n, int nslice, int block,
                  StepParams p) {
    extern __shared__ float4 sx[];
    __shared__ double red[16][kDiagFields];
    const int4 ch = chunks[blockIdx.x];
    const int b = ch.x, base = b * block;
    const int t = threadIdx.x;
    const int own = lane_mass[base + t];
    const int h0 = halo_ptr[b], h1 = halo_ptr[b + 1];
    float4 xt = xin[min(base + t, n - 1)];
    const int s = __builtin_amdgcn_readfirstlane((base + t) >> 6);
    const int e0 = __builtin_amdgcn_readfirstlane(slice_ptr[min(s, nslice - 1)]);
    const int w = s < nslice ? __builtin_amdgcn_readfirstlane((slice_ptr[min(s, nslice - 1) + 1] - e0) >> 6) : 0;
    int slot[4], g[4];
    float2 c[4];
    auto fetch = [&](int r) {   // past the end: the last row again (an empty slice: the arrays' padding)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + max(min(r + u, w - 1), 0) * 64 + (t & 63);
            slot[u] = nbr[e];
            c[u] = kl[e];
            g[u] = ACT ? (int)grp[e] : 0;
        }
    };
    fetch(0);
    xt.w = __int_as_float(base + t);
    sx[t] = xt;
    for (int q = h0 + t; q < h1; q += block) {
        const int j = halo_idx[q];
        float4 xh = xin[j];
        xh.w = __int_as_float(j);
        sx[block + (q - h0)] = xh;
    }
    __syncthreads();
    const float4 xi = sx[own];
    const int i = base + own;
    const bool mine = i >= ch.y && i < ch.z;
    // fields: 0 ke, 1 pe_spring, 2 pe_grav, 3 pe_contact, 4-6 momentum, 7-9 sum m x,
    //         10 mass, 11-13 bbox max, 14-16 bbox min, 17 non-finite count
    double acc[18];
    for (int f = 0; f < 11; ++f) acc[f] = 0.0;
    acc[11] = acc[12] = acc[13] = -1e300;
    acc[14] = acc[15] = acc[16] = 1e300;
    acc[17] = 0.0;
    if (mine) {
        const double m = mass[i];
        const double x = (double)xi.x + p.ox, y = (double)xi.y + p.oy, z = (double)xi.z + p.oz;
        const double vx = vin[3 * i], vy = vin[3 * i + 1], vz = vin[3 * i + 2];
        acc[0] = 0.5 * m * (vx * vx + vy * vy + vz * vz);
        acc[2] = -m * ((double)p.gx * x + (double)p.gy * y + (double)p.gz * z);
        if (p.ground) {
            const double pen = (double)p.ground_z - (double)xi.z;   // both in device coordinates
            if (pen > 0.0) acc[3] = 0.5 * (double)p.ground_k * pen * pen;
        }
        acc[4] = m * vx; acc[5] = m * vy; acc[6] = m * vz;
        acc[7] = m * x;  acc[8] = m * y;  acc[9] = m * z;
        acc[10] = m;
        acc[11] = x; acc[12] = y; acc[13] = z;
        acc[14] = x; acc[15] = y; acc[16] = z;
        const bool fin = isfinite(x) && isfinite(y) && isfinite(z) && isfinite(vx) && isfinite(vy) && isfinite(vz);
        acc[17] = fin ? 0.0 : 1.0;
    }
    // spring energy of springs whose other end has a larger index
    double es = 0.0;
    for (int r = 0; r < w; r += 4) {
        double term[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            double l0 = (double)c[u].y;
            if (ACT) l0 *= (double)factor[g[u]];
            const float4 xj = sx[slot[u]];
            const double dx = (double)xj.x - (double)xi.x, dy = (double)xj.y - (double)xi.y,
                         dz = (double)xj.z - (double)xi.z;
            const double dl = sqrt(dx * dx + dy * dy + dz * dz) - l0;
            term[u] = r + u < w && __float_as_int(xj.w) > i ? 0.5 * (double)c[u].x * dl * dl : 0.0;
        }
        if (r + 4 < w) fetch(r + 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) es += term[u];
    }
    if (mine) acc[1] = es;
    const int wv = t >> 6, nw = (blockDim.x + 63) >> 6;
    double r[18];
    for (int f = 0; f < 11; ++f) r[f] = wave_sum(acc[f]);
    for (int f = 11; f < 14; ++f) r[f] = wave_max(acc[f]);
    for (int f = 14; f < 17; ++f) r[f] = wave_min(acc[f]);
    r[17] = wave_sum(acc[17]);
    if ((t & 63) == 0)
        for (int f = 0; f < 18; ++f) red[wv][f] = r[f];
    __syncthreads();
    if (t == 0) {
        double o[18];
        for (int f = 0; f < 18; ++f) o[f] = red[0][f];
        for (int w2 = 1; w2 < nw; ++w2) {
            for (int f = 0; f < 11; ++f) o[f] += red[w2][f];
            for (int f = 11; f < 14; ++f) o[f] = fmax(o[f], red[w2][f]);
            for (int f = 14; f < 17; ++f) o[f] = fmin(o[f], red[w2][f]);
            o[17] += red[w2][17];
        }
        double* out = part + (size_t)blockIdx.x * kDiagFields;
        for (int f = 0; f < 18; ++f) out[f] = o[f];
    }
}

// Per body: its chunks' partial results, one wavefront per body, each lane over every 64th chunk in
// order, then across the lanes (a fixed order, independent of the launch's shape; one thread per body
// would walk the 1,250 chunks of 640,000 masses one latency after the other).  `out` is pinned host memory.
__global__ void __launch_bounds__(64)
diag_body_kernel(const double* __restrict__ part, const int32_t* __restrict__ body_chunk, double* __restrict__ out) {
    const int bdy = (int)blockIdx.x, lane = (int)threadIdx.x;
    const int c1 = body_chunk[bdy + 1];
    double o[18];
    for (int f = 0; f < 18; ++f) o[f] = (f >= 11 && f < 14) ? -1e300 : (f >= 14 && f < 17 ? 1e300 : 0.0);
    for (int c = body_chunk[bdy] + lane; c < c1; c += 64) {
        const double* q = part + (size_t)c * kDiagFields;
        for (int f = 0; f < 11; ++f) o[f] += q[f];
        for (int f = 11; f < 14; ++f) o[f] = fmax(o[f], q[f]);
        for (int f = 14; f < 17; ++f) o[f] = fmin(o[f], q[f]);
        o[17] += q[17];
    }
    for (int f = 0; f < 18; ++f) {
        const double v = f >= 11 && f < 14 ? wave_max(o[f]) : f >= 14 && f < 17 ? wave_min(o[f]) : wave_sum(o[f]);
        if (lane == 0) out[(size_t)bdy * kDiagFields + f] = v;
    }
}

// ---------------------------------------------------------------- adjoint of one step
//
// For the loss L = sum_i w_i . x_i(T), with (x_bar', v_bar') the adjoints of the outputs of
// step n, the reverse of the step is (see the step above, in reverse order):
//   v'_bar_tot = v_bar' + dt x_bar'          (x' = x + dt v')
//   v**_bar    = (1 - d) v'_bar_tot          (damping)
//   v*_bar     = J^T v**_bar                 (friction clamp: J = I - (c/|v_t|)(I - u u^T) on
//                                             the tangential part when sliding, 0 when stuck)
//   c_bar      = -u . v**_bar_t,  c = mu k_g (z_g - z) dt / m  ->  z_bar += c_bar (-mu k_g dt / m)
//   w          = dt v*_bar / m               (adjoint of the force on the mass)
//   x_bar      = x_bar' - k_g w_z (contact) + sum_springs K_s (w_j - w_i)
//   K_s        = k [n n^T + (delta / l)(I - n n^T)]
//   theta_bar += (dL0/dtheta) k n . (w_j - w_i)   (actuated springs)
// Fixed masses (1/m = 0) have w = 0 and v_bar = 0.  adj_local computes everything but the
// spring sum; adj_gather adds the spring sum with the same LDS-staged incidence walk as the
// step, and accumulates each actuated spring's sensitivity in FP64, half from each end.

// adj_local for mass i, given its x_bar' (bx, by, bz); v_bar', the position and v* are loaded apart,
// so that a caller can do so early.
struct AdjLocalIn {
    float4 x;
    float vb[3], vs[2];
    __device__ __forceinline__ void load(int i, const float4* __restrict__ px, const float* __restrict__ vstar,
                                         const float* __restrict__ vb1) {
        x = px[i];
        for (int c = 0; c < 3; ++c) vb[c] = vb1[3 * i + c];
        for (int c = 0; c < 2; ++c) vs[c] = vstar[3 * i + c];
    }
};

__device__ __forceinline__ void adj_local_one(int i, const AdjLocalIn& in, float bx, float by, float bz,
                                              float4* __restrict__ w, float* __restrict__ vb0,
                                              float* __restrict__ xbl, const StepParams& p) {
    const float4 xi = in.x;
    const float inv_m = xi.w;
    const float tx = __builtin_fmaf(p.dt, bx, in.vb[0]);
    const float ty = __builtin_fmaf(p.dt, by, in.vb[1]);
    const float tz = __builtin_fmaf(p.dt, bz, in.vb[2]);
    float gx = p.damp * tx, gy = p.damp * ty, gz = p.damp * tz;
    float zb = 0.0f;
    float wz_contact = 0.0f;
    if (inv_m == 0.0f) {
        w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        vb0[3 * i + 0] = vb0[3 * i + 1] = vb0[3 * i + 2] = 0.0f;
        xbl[3 * i + 0] = bx;
        xbl[3 * i + 1] = by;
        xbl[3 * i + 2] = bz;
        return;
    }
    const float pen = p.ground ? p.ground_z - xi.z : 0.0f;
    const bool touching = pen > 0.0f;
    if (touching) {
        const float fn = p.ground_k * pen;
        const float c = p.ground_mu * fn * p.dt * inv_m;
        const float vx = in.vs[0], vy = in.vs[1];
        const float sp = __builtin_sqrtf(vx * vx + vy * vy);
        if (sp > c) {
            const float ux = vx / sp, uy = vy / sp;
            const float ug = ux * gx + uy * gy;
            const float r = c / sp;
            gx = gx - r * (gx - ux * ug);
            gy = gy - r * (gy - uy * ug);
            zb = -ug * (-p.ground_mu * p.ground_k * p.dt * inv_m);
        } else {
            gx = gy = 0.0f;
        }
    }
    const float wx = p.dt * gx * inv_m, wy = p.dt * gy * inv_m, wz = p.dt * gz * inv_m;
    if (touching) wz_contact = -p.ground_k * wz;
    w[i] = make_float4(wx, wy, wz, 0.0f);
    vb0[3 * i + 0] = gx;
    vb0[3 * i + 1] = gy;
    vb0[3 * i + 2] = gz;
    xbl[3 * i + 0] = bx;
    xbl[3 * i + 1] = by;
    xbl[3 * i + 2] = bz + wz_contact + zb;
}

__global__ void __launch_bounds__(256)
adj_local_kernel(const float4* __restrict__ x, const float* __restrict__ vstar, const float* __restrict__ xb1,
                 const float* __restrict__ vb1, float4* __restrict__ w, float* __restrict__ vb0,
                 float* __restrict__ xbl, int n, StepParams p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    AdjLocalIn in;
    in.load(i, x, vstar, vb1);
    adj_local_one(i, in, xb1[3 * i + 0], xb1[3 * i + 1], xb1[3 * i + 2], w, vb0, xbl, p);
}

// Where the sensitivities of actuated springs (FP64) go.  kAdjBlockSums: every lane sums its springs'
// in a column of LDS of its own, one row per actuation group of the workgroup's range; the columns
// are then added in a fixed order and the workgroup's sums, not each entry's, cross the launches.
// kAdjEntrySums (ranges too wide for that, see adj_block_sums): one sum per entry in memory, read and
// written by every launch, 32 of the 44 bytes an entry then costs.  Block against entry sums: the
// quadruped's launch 7.0 against 8.5 us and the sums at the end 2 against 48; 60 reversed steps of 32
// robots (239k masses) 3.9 against 4.5 ms.
enum : int { kAdjPassive = 0, kAdjEntrySums = 1, kAdjBlockSums = 2 };

struct AdjArgs {
    const float4* __restrict__ x;
    const float4* __restrict__ w;
    const float* __restrict__ xbl;
    float* __restrict__ xb0;
    const int32_t* __restrict__ slice_ptr;
    const uint16_t* __restrict__ nbr;
    const float2* __restrict__ kl;
    const uint16_t* __restrict__ grp;
    const int32_t* __restrict__ halo_ptr;
    const int32_t* __restrict__ halo_idx;
    const uint16_t* __restrict__ lane_mass;
    const float* __restrict__ factor;
    double2* __restrict__ sens;
    const int4* __restrict__ range;   // kAdjBlockSums: (first group, groups, first sum) of each block
    double cos_t, sin_t;
    int n_factor, n, nblk, nslice, block, lds_slots;
    int max_groups;      // kAdjBlockSums: of any block
    int stage_factors;   // kAdjEntrySums: the factor table goes through LDS (small tables: no dependent global load)
};

// What an entry holds for the reverse step: neighbour slot, (k, L0), the index of its factor and, with
// kAdjEntrySums, the sensitivity summed so far.
typedef float adj_pair __attribute__((ext_vector_type(2)));
typedef double adj_sum __attribute__((ext_vector_type(2)));
template <int MODE>
struct AdjEntry {
    uint32_t slot, g;
    adj_pair kl;
    adj_sum acc;
};

template <int MODE>
__device__ __forceinline__ AdjEntry<MODE> adj_entry(const AdjArgs& a, int e) {
    AdjEntry<MODE> q;
    q.slot = a.nbr[e];
    q.kl = reinterpret_cast<const adj_pair*>(a.kl)[e];
    q.g = MODE != kAdjPassive ? (uint32_t)a.grp[e] : (uint32_t)a.n_factor;
    if (MODE == kAdjEntrySums) q.acc = reinterpret_cast<const adj_sum*>(a.sens)[e];
    return q;
}

// A workgroup's actuation factors and sums, after its positions and adjoint forces in LDS.
template <int MODE>
struct AdjGroups {
    double* column;   // kAdjBlockSums: this thread's, a row of `threads` apart per group
    float* factor;
    int first, count, slot, threads;
    adj_sum old;      // the sum that this lane will add to
    float early;

    // Sixteen lanes add up a row, so that all rows of a usual range go at once; the first of them
    // stores it.  (A wavefront per row, the rows one after the other, cost 1 us at the launch's end.)
    __device__ __forceinline__ int pitch() const { return threads + 16; }   // rows apart in the banks
    __device__ __forceinline__ void start(const AdjArgs& a, float4* lds, int b) {
        threads = (int)blockDim.x;
        if (MODE == kAdjEntrySums) factor = reinterpret_cast<float*>(lds);
        if (MODE == kAdjBlockSums) {
            const int4 r = a.range[b];
            first = r.x;
            count = r.y;
            slot = r.z;
            column = reinterpret_cast<double*>(lds) + threadIdx.x;
            factor = reinterpret_cast<float*>(reinterpret_cast<double*>(lds) + (a.max_groups + 1) * pitch());
            const int q = (int)threadIdx.x >> 4;
            if ((threadIdx.x & 15u) == 0 && q < count) old = reinterpret_cast<const adj_sum*>(a.sens)[slot + q];
            if ((int)threadIdx.x < count) early = a.factor[first + (int)threadIdx.x];
        }
    }
    // what start loaded, into LDS
    __device__ __forceinline__ void stage(const AdjArgs& a) {
        if (MODE == kAdjBlockSums) {
            if ((int)threadIdx.x < count) factor[threadIdx.x] = early;
            for (int q = (int)threadIdx.x + threads; q < count; q += threads) factor[q] = a.factor[first + q];
            for (int q = 0; q < count; ++q) column[q * pitch()] = 0.0;
        } else if (MODE == kAdjEntrySums) {
            if (a.stage_factors)
                for (int q = (int)threadIdx.x; q <= a.n_factor; q += threads) factor[q] = a.factor[q];
        }
    }
    // the factor of an entry's rest length (after the barrier)
    __device__ __forceinline__ float of(const AdjArgs& a, uint32_t g) const {
        if (MODE == kAdjPassive) return 1.0f;
        if (MODE == kAdjBlockSums) return g < (uint32_t)a.n_factor ? factor[(int)g - first] : 1.0f;
        if (a.stage_factors) return factor[g];   // LDS and global memory apart: one pointer to either is a flat load
        return a.factor[g];
    }
    // s counts where `use` is set and the spring is actuated
    __device__ __forceinline__ void add(const AdjArgs& a, int e, uint32_t g, adj_sum acc, bool use, double s) {
        use = use && g < (uint32_t)a.n_factor;
        if (MODE == kAdjBlockSums) {
            // one lane per column, so the order is the lane's own; the row after the last takes what does not count
            typedef __attribute__((address_space(3))) double* lds_double;
            (void)__builtin_amdgcn_ds_atomic_fadd_f64((lds_double)(column + (use ? (int)g - first : count) * pitch()), s);
        } else if (use) {
            acc.x += a.cos_t * s;
            acc.y += a.sin_t * s;
            reinterpret_cast<adj_sum*>(a.sens)[e] = acc;
        }
    }
    // every thread of the workgroup
    __device__ __forceinline__ void finish(const AdjArgs& a) {
        if (MODE != kAdjBlockSums) return;
        __syncthreads();
        const int part = (int)(threadIdx.x & 15u), per = threads >> 4;
        const double* rows = column - threadIdx.x;
        for (int r0 = 0; r0 < count; r0 += per) {
            const int r = r0 + ((int)threadIdx.x >> 4);
            double v = 0.0;
            if (r < count)
                for (int c = part; c < threads; c += 16) v += rows[r * pitch() + c];
            v += dpp_double<0xB1>(v);    // lane ^ 1
            v += dpp_double<0x4E>(v);    // lane ^ 2
            v += dpp_double<0x141>(v);   // the other half of eight
            v += dpp_double<0x140>(v);   // the other half of sixteen
            if (part == 0 && r < count) {
                adj_sum* to = reinterpret_cast<adj_sum*>(a.sens) + slot + r;
                adj_sum now = r0 ? *to : old;
                now.x += a.cos_t * v;
                now.y += a.sin_t * v;
                *to = now;
            }
        }
    }
};

// One incidence: the spring's tangent stiffness applied to w_j - w_i, and (actuated) the sensitivity
// of the loss to its rest length, accumulated in FP64.
template <int MODE>
__device__ __forceinline__ void adj_spring(const AdjArgs& a, AdjGroups<MODE>& groups, int e, const AdjEntry<MODE>& q,
                                           float f, bool ok, float4 xi, float4 wi, lds_vec4 xj, lds_vec4 wj, float& ax,
                                           float& ay, float& az) {
    const float l0 = MODE != kAdjPassive ? q.kl.y * f : q.kl.y;
    const float dx = xj.x - xi.x, dy = xj.y - xi.y, dz = xj.z - xi.z;
    const float len2 = dx * dx + dy * dy + dz * dz;
    const bool use = ok && len2 > 0.0f;   // selects, not a branch: the rows of a lane then overlap
    const float len = __builtin_sqrtf(use ? len2 : 1.0f);
    const float il = 1.0f / len;
    const float nx = dx * il, ny = dy * il, nz = dz * il;
    const float dwx = wj.x - wi.x, dwy = wj.y - wi.y, dwz = wj.z - wi.z;
    const float ndw = nx * dwx + ny * dwy + nz * dwz;
    const float tr = 1.0f - l0 * il;        // delta / l
    const float k = q.kl.x;
    const float sx = ax + k * (nx * ndw + tr * (dwx - nx * ndw));
    const float sy = ay + k * (ny * ndw + tr * (dwy - ny * ndw));
    const float sz = az + k * (nz * ndw + tr * (dwz - nz * ndw));
    ax = use ? sx : ax;
    ay = use ? sy : ay;
    az = use ? sz : az;
    if (MODE != kAdjPassive) groups.add(a, e, q.g, q.acc, use, 0.5 * (double)q.kl.y * (double)k * (double)ndw);
}

__device__ __forceinline__ lds_vec4 vec4_of(float4 v) {
    const lds_vec4 r = {v.x, v.y, v.z, v.w};
    return r;
}

// The step reversed, one lane per mass (bodies that fill the chip by themselves).  With nx.x set, the
// mass's x_bar then feeds adj_local of the step before (every input of which is the mass's own), so
// one launch per reversed step remains; nx.w and nx.xbl must not be the w and xbl this launch reads.
// (x_bar itself is then needed by nobody else.)
template <int MODE>
__global__ void __launch_bounds__(1024) adj_gather_kernel(AdjArgs a, StepParams p, AdjNext nx) {
    extern __shared__ float4 sx[];
    float4* sw = sx + a.lds_slots;
    const int b = logical_block(a.nblk);
    if (b >= a.nblk) return;
    const int base = b * a.block, t = (int)threadIdx.x;
    AdjGroups<MODE> groups;
    groups.start(a, sw + a.lds_slots, b);
    groups.stage(a);
    float4 wt = make_float4(0.f, 0.f, 0.f, 0.f);
    if (base + t < a.n) wt = a.w[base + t];
    sw[t] = wt;
    const int h0 = a.halo_ptr[b], h1 = a.halo_ptr[b + 1];
    for (int h = h0 + t; h < h1; h += a.block) sw[a.block + (h - h0)] = a.w[a.halo_idx[h]];
    const int own = stage_positions(sx, a.x, a.halo_ptr, a.halo_idx, a.lane_mass, b, base, a.n, a.block);
    const float4 xi = sx[own];
    const float4 wi = sw[own];
    float ax = 0.f, ay = 0.f, az = 0.f;
    const int s = __builtin_amdgcn_readfirstlane((base + t) >> 6);
    if (s < a.nslice) {
        const int e0 = __builtin_amdgcn_readfirstlane(a.slice_ptr[s]);
        const int rows = __builtin_amdgcn_readfirstlane((a.slice_ptr[s + 1] - e0) >> 6);
        const int e = e0 + (t & 63);
        constexpr int B = 8;   // rows whose loads are in flight together
        int k = 0;
        for (; k + B <= rows; k += B) {
            AdjEntry<MODE> q[B];
            float f[B];
#pragma unroll
            for (int u = 0; u < B; ++u) q[u] = adj_entry<MODE>(a, e + (k + u) * 64);
#pragma unroll
            for (int u = 0; u < B; ++u) f[u] = groups.of(a, q[u].g);
#pragma unroll
            for (int u = 0; u < B; ++u)
                adj_spring<MODE>(a, groups, e + (k + u) * 64, q[u], f[u], true, xi, wi, vec4_of(sx[q[u].slot]), vec4_of(sw[q[u].slot]),
                                ax, ay, az);
        }
        for (; k < rows; ++k) {
            const AdjEntry<MODE> q = adj_entry<MODE>(a, e + k * 64);
            adj_spring<MODE>(a, groups, e + k * 64, q, groups.of(a, q.g), true, xi, wi, vec4_of(sx[q.slot]),
                             vec4_of(sw[q.slot]), ax, ay, az);
        }
    }
    const int i = base + own;
    if (i < a.n) {
        const float bx = a.xbl[3 * i + 0] + ax, by = a.xbl[3 * i + 1] + ay, bz = a.xbl[3 * i + 2] + az;
        if (nx.x) {
            AdjLocalIn in;
            in.load(i, nx.x, nx.vstar, nx.vb1);
            adj_local_one(i, in, bx, by, bz, nx.w, nx.vb0, nx.xbl, p);
        } else {
            a.xb0[3 * i + 0] = bx;
            a.xb0[3 * i + 1] = by;
            a.xb0[3 * i + 2] = bz;
        }
    }
    groups.finish(a);
}

// The same with LPM lanes per mass (2 or 4; the simulation's lanes per mass): lane j of a mass takes its
// incidence rows j, j + LPM, ... and the partial sums are combined by the same fixed cross-lane
// pairing as the step's; each incidence's sensitivity is still accumulated by exactly one lane.
// Such a launch is a chain of latencies (the quadruped: under one wavefront per SIMD), so every load
// is issued as early as it can be: the first kAdjPre rows of each lane (at four lanes all rows of a
// full lattice's masses), the halo, and what adj_local needs, before anything is waited for.
// The quadruped's launch: 9.7 -> 7.0 us beside the recomputed steps (7.8 -> 6.0 alone).
constexpr int kAdjPre = 8, kAdjGroup = 4;

template <int MODE, int LPM>
__global__ void __launch_bounds__(1024) adj_gather_lanes_kernel(AdjArgs a, StepParams p, AdjNext nx) {
    extern __shared__ float4 sx[];
    float4* sw = sx + a.lds_slots;
    const int b = logical_block(a.nblk);
    if (b >= a.nblk) return;
    const int t = (int)threadIdx.x, nt = (int)blockDim.x, base = b * a.block;
    const int m = t / LPM, sub = t % LPM;
    const int h0 = a.halo_ptr[b], h1 = a.halo_ptr[b + 1];
    const int own = a.lane_mass[base + m];
    const int hj = h0 + t < h1 ? a.halo_idx[h0 + t] : -1;
    // no condition around these loads, only clamped addresses: after a load that may be skipped, the next
    // wait is for every load
    const int it = min(base + min(t, a.block - 1), a.n - 1);
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 xt = a.x[it], wt = a.w[it], xh = z, wh = z;
    // this lane's rows: sub, sub + LPM, ...; the slice's last row can be missing in some lanes of a group
    const int s = __builtin_amdgcn_readfirstlane((base + m) >> 6);
    int e = 0, rows = 0, count = 0;
    if (s < a.nslice) {
        const int e0 = __builtin_amdgcn_readfirstlane(a.slice_ptr[s]);
        rows = __builtin_amdgcn_readfirstlane((a.slice_ptr[s + 1] - e0) >> 6);
        count = (rows + LPM - 1) / LPM;
        e = e0 + (m & 63);
    }
    auto at = [&](int k) { return e + max(min(k * LPM + sub, rows - 1), 0) * 64; };   // past the end: the last row again
    AdjEntry<MODE> q[kAdjPre];
#pragma unroll
    for (int u = 0; u < kAdjPre; ++u) q[u] = adj_entry<MODE>(a, at(u));   // (an empty slice: the arrays' padding)
    if (hj >= 0) {
        xh = a.x[hj];
        wh = a.w[hj];
    }
    AdjGroups<MODE> groups;
    groups.start(a, sw + a.lds_slots, b);
    if (base + t >= a.n) xt = wt = z;
    const int i = base + own;
    const bool mine = sub == 0 && i < a.n;
    AdjLocalIn in = {};
    float xb[3] = {};
    if (mine) {
        for (int c = 0; c < 3; ++c) xb[c] = a.xbl[3 * i + c];
        if (nx.x) in.load(i, nx.x, nx.vstar, nx.vb1);
    }
    groups.stage(a);
    if (t < a.block) {   // block * LPM threads: one round
        sx[t] = xt;
        sw[t] = wt;
    }
    if (hj >= 0) {
        sx[a.block + t] = xh;
        sw[a.block + t] = wh;
    }
    for (int h = h0 + t + nt; h < h1; h += nt) {
        const int j = a.halo_idx[h];
        sx[a.block + (h - h0)] = a.x[j];
        sw[a.block + (h - h0)] = a.w[j];
    }
    __syncthreads();
    const float4 xi = sx[own], wi = sw[own];
    float ax = 0.f, ay = 0.f, az = 0.f;
    // N rows from row k on, their LDS reads together
    auto part = [&](auto rows_of, const AdjEntry<MODE>* g, int k) {
        constexpr int N = decltype(rows_of)::value;
        lds_vec4 xj[N], wj[N];
        float f[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            xj[u] = vec4_of(sx[g[u].slot]);
            wj[u] = vec4_of(sw[g[u].slot]);
            f[u] = groups.of(a, g[u].g);
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
            adj_spring<MODE>(a, groups, e + ((k + u) * LPM + sub) * 64, g[u], f[u], (k + u) * LPM + sub < rows, xi, wi,
                             xj[u], wj[u], ax, ay, az);
    };
    auto group = [&](const AdjEntry<MODE>* g, int k) {   // up to kAdjGroup rows; the count is uniform
        switch (min(count - k, kAdjGroup)) {
        case 1: part(std::integral_constant<int, 1>{}, g, k); break;
        case 2: part(std::integral_constant<int, 2>{}, g, k); break;
        case 3: part(std::integral_constant<int, 3>{}, g, k); break;
        case 4: part(std::integral_constant<int, 4>{}, g, k); break;
        }
    };
    static_assert(kAdjGroup == 4, "the cases above");
#pragma unroll
    for (int u = 0; u < kAdjPre; u += kAdjGroup)
        if (u < count) group(q + u, u);
    for (int k = kAdjPre; k < count; k += kAdjGroup) {
#pragma unroll
        for (int u = 0; u < kAdjGroup; ++u) q[u] = adj_entry<MODE>(a, at(k + u));
        group(q, k);
    }
#pragma unroll
    for (int o = 1; o < LPM; o <<= 1) {
        ax += __shfl_xor(ax, o, 64);
        ay += __shfl_xor(ay, o, 64);
        az += __shfl_xor(az, o, 64);
    }
    if (mine) {
        const float bx = xb[0] + ax, by = xb[1] + ay, bz = xb[2] + az;
        if (nx.x) {
            adj_local_one(i, in, bx, by, bz, nx.w, nx.vb0, nx.xbl, p);
        } else {
            a.xb0[3 * i + 0] = bx;
            a.xb0[3 * i + 1] = by;
            a.xb0[3 * i + 2] = bz;
        }
    }
    groups.finish(a);
}

// ---------------------------------------------------------------------------------------
// Structured-box form (the lattice of section "Generating a Lattice" filled out to a full
// box): every node of an nx x ny x nz grid is a mass, every pair of grid neighbours (the 26
// directions) is a spring, the rest length depends only on the kind of direction (edge, face
// diagonal, body diagonal), and the stiffness on the direction and on which faces of the box
// the mass lies on (27 boundary classes; interior masses: on the kind only).  The
// host detects this structure (cronos_create) and then no incidence data is read at all: a
// workgroup owns one aligned 8 x 8 x 8 cube of the Morton order (512 masses, 512 threads),
// stages it with a one-node halo as a 10 x 10 x 10 tile in LDS, and each lane visits its 26
// tile neighbours at fixed offsets.  Directions are summed in a fixed order (dz, dy, dx
// ascending), so the result is bitwise reproducible; it equals the other forms' CSR-order
// sum to rounding.  Halo cells outside the box hold a far-away position whose spring has
// k = 0, contributing exactly nothing.
constexpr int kGridEdge = 8, kGridPitch = 10, kGridCells = 1000, kGridHalo = 488, kGridThreads = 512;

struct GridArgs {
    const float4* __restrict__ xin;
    const float* __restrict__ vin;
    float4* __restrict__ xout;
    float* __restrict__ vout;
    float* __restrict__ vstar_out;
    const float* __restrict__ fext;
    const int32_t* __restrict__ halo;   // [nblk][kGridHalo] new index of each halo cell, -1 outside
    const int4* __restrict__ org;       // [nblk] grid coordinates of the block's first node
    const float* __restrict__ kcls;     // [27][26] k per (boundary class, direction)
    const uint32_t* __restrict__ tab;   // [512] lane's tile cell | lx << 10 | ly << 13 | lz << 16,
                                        // then [488] tile cell of each halo slot
    int nblk, nx, ny, nz;
    // per direction kind (edge, face diagonal, body diagonal: 1, 2 or 3 non-zero offsets)
    float kin[3];                       // k of interior masses (class 13)
    float l0[3];                        // rest length
    double q[3];                        // its square, exact in FP64
};

// Sum of the 26 spring forces of the lane's mass at tile cell `cell`.  INTERIOR: every mass of
// the wavefront is interior, so each direction's k is the same for all lanes.
template <int EX, bool INTERIOR>
__device__ __forceinline__ void gather_grid(const float4* __restrict__ tile, const float* __restrict__ kc, int cell,
                                            float4 xi, const GridArgs& a, float& fx, float& fy, float& fz) {
    fx = fy = fz = 0.0f;
#pragma unroll
    for (int d = 0; d < 26; ++d) {
        const int e = d < 13 ? d : d + 1;                 // skip the centre of the 3 x 3 x 3 stencil
        const int ox = e % 3 - 1, oy = (e / 3) % 3 - 1, oz = e / 9 - 1;
        const int kind = (ox != 0) + (oy != 0) + (oz != 0) - 1;
        const float4 xj = tile[cell + (oz * kGridPitch + oy) * kGridPitch + ox];
        const float k = INTERIOR ? a.kin[kind] : kc[d];
        float dx, dy, dz;
        const float fac = hooke_fac<EX>(xi.x, xi.y, xi.z, xj.x, xj.y, xj.z, k, a.l0[kind], a.q[kind], dx, dy, dz);
        fx = __builtin_fmaf(fac, dx, fx);
        fy = __builtin_fmaf(fac, dy, fy);
        fz = __builtin_fmaf(fac, dz, fz);
    }
}

template <bool EXACT>
__global__ void __launch_bounds__(kGridThreads) step_grid_kernel(GridArgs a, StepParams p) {
    __shared__ float4 tile[kGridCells];
    __shared__ float kcls[27 * 26];
    const int b = logical_block(a.nblk);
    if (b >= a.nblk) return;
    const int t = threadIdx.x;
    const int i = b * kGridThreads + t;
    const uint32_t lane_info = a.tab[t];      // the block's mass t: its tile cell and local x, y, z
    const int cell = (int)(lane_info & 1023u);
    const float4 xi = a.xin[i];
    tile[cell] = xi;
    for (int h = t; h < kGridHalo; h += kGridThreads) {
        const int g = a.halo[(long)b * kGridHalo + h];
        tile[a.tab[kGridThreads + h]] = g >= 0 ? a.xin[g] : make_float4(1e18f, 1e18f, 1e18f, 0.0f);
    }
    // a block that touches no face of the box holds only interior masses (class 13): it needs
    // neither the class of each mass nor the per-class k table
    const int4 o = a.org[b];
    const bool face = o.x == 0 || o.y == 0 || o.z == 0 || o.x + kGridEdge >= a.nx || o.y + kGridEdge >= a.ny ||
                      o.z + kGridEdge >= a.nz;
    int cls = 13;
    if (face) {
        for (int q = t; q < 27 * 26; q += kGridThreads) kcls[q] = a.kcls[q];
        const int gx = o.x + (int)((lane_info >> 10) & 7u), gy = o.y + (int)((lane_info >> 13) & 7u),
                  gz = o.z + (int)((lane_info >> 16) & 7u);
        cls = (gx == 0 ? 0 : gx == a.nx - 1 ? 2 : 1) + 3 * (gy == 0 ? 0 : gy == a.ny - 1 ? 2 : 1) +
              9 * (gz == 0 ? 0 : gz == a.nz - 1 ? 2 : 1);
    }
    __syncthreads();
    const float* kc = kcls + 26 * cls;
    const bool interior = __builtin_amdgcn_ballot_w64(cls != 13) == 0;
    const int mode = EXACT ? difference_mode(xi, p.safe) : kPlain;
    float fx, fy, fz;
    if (mode == kPlain) {
        if (interior) gather_grid<kPlain, true>(tile, kc, cell, xi, a, fx, fy, fz);
        else gather_grid<kPlain, false>(tile, kc, cell, xi, a, fx, fy, fz);
    } else if (mode == kExactZ) {
        if (interior) gather_grid<kExactZ, true>(tile, kc, cell, xi, a, fx, fy, fz);
        else gather_grid<kExactZ, false>(tile, kc, cell, xi, a, fx, fy, fz);
    } else {
        if (interior) gather_grid<kExactAll, true>(tile, kc, cell, xi, a, fx, fy, fz);
        else gather_grid<kExactAll, false>(tile, kc, cell, xi, a, fx, fy, fz);
    }
    float vx = a.vin[3 * i + 0], vy = a.vin[3 * i + 1], vz = a.vin[3 * i + 2];
    float4 xo;
    integrate(p, p.dtv, xi, fx, fy, fz, a.fext ? a.fext + 3 * i : nullptr, vx, vy, vz, xo,
              a.vstar_out ? a.vstar_out + 3 * i : nullptr);
    a.xout[i] = xo;
    a.vout[3 * i + 0] = vx;
    a.vout[3 * i + 1] = vy;
    a.vout[3 * i + 2] = vz;
}

inline int grid_for(int64_t nblk) { return (int)(((nblk + 7) / 8) * 8); }

constexpr int kAdjStagedFactors = 4096;

// Explicit bodies of 64-mass workgroups up to this size take four lanes per mass.  One lane against four:
// 1,000 masses 5.35 / 4.50 us a step, 4,320 5.2 / 4.3, 12,711 7.95 / 6.72, 18,000 5.31 / 5.20, 24,000
// 5.67 / 5.68, 48,400 5.74 / 6.17 (above some 16,000 masses the SIMDs hold several wavefronts, and the
// sums that every lane repeats are no longer free); workgroups of 256 masses, 1,000: 5.04 / 7.69.
// Fewer than six entry rows a mass are not worth it (300 masses, one lane against four: no springs 1.87 / 2.34,
// 2 rows 2.60 / 2.75, 4 rows 2.85 / 2.78, 8 rows 3.28 / 3.05, 26 rows 5.16 / 4.40).
constexpr int64_t kQuadMasses = 16384;
constexpr float kQuadRows = 6.0f;

int step_mode(const DeviceArrays& d) { return d.sp_rec ? kSplit : d.narrow ? kNarrow : d.packed ? kTable : kExplicit; }

// Entries that a one-lane step keeps in flight.  Two at a time are left to the forms that gain by them: compact
// entries are loaded a batch ahead, and a batch of two is then too short to hide anything (26 rows a mass, two
// against four: 1,000 masses 6.05 / 4.83 us, 400,000 16.45 / 14.56); passive explicit entries run four
// either way (5.58 / 4.92 and 21.5 / 21.6), and so do passive split ones (28.7 /
// 25.9).  The springs are added in row order whatever it is.
int step_batch(const DeviceArrays& d, int mode) {
    return d.batch == 2 && !(d.grp && (mode == kSplit || mode == kExplicit)) ? 4 : d.batch;
}

bool quads(const DeviceArrays& d) { return d.block == 64 && d.n <= kQuadMasses && d.mean_rows >= kQuadRows; }

// Several lanes per mass with their entries loaded up front, and every LDS read of eight rows before the first
// spring (lane_early): 64-110 registers against 27-52, and up to a row more than a slice has.  That pays where
// wavefronts are alone on their SIMDs (all of them together at most one for each of the 1024, in workgroups
// of at most four) and each lane has several rows; else rows go in pairs (lane_pairs), with the same sums.
// Pairs / up front, us a step, 26 rows a mass: 4 lanes in 64-mass workgroups 1,000 masses 3.87 / 3.49, 12,000
// 4.05 / 3.64, 24,000 4.22 / 4.37, 120,000 7.65 / 8.62; 2 lanes 24,000 5.50 / 5.19, 60,000 5.98 / 6.00;
// workgroups of 512 threads 12,000 4.16 / 4.40, of 1024 threads 4.79 / 5.30 (4 lanes), 6.17 / 7.25 (2).  Fewer
// rows (4 lanes, 64-mass workgroups, 12,000 masses): 14 rows 3.46 / 3.44, 8 rows 3.08 / 3.36, 2 rows 2.89 / 3.25.
bool lanes_early(const DeviceArrays& d) {
    return d.block * d.lanes <= 256 && d.n * d.lanes <= 64 * 1024 && d.mean_rows >= 5.0f * (float)d.lanes;
}

// LDS that a workgroup may take for kAdjBlockSums: what a launch may have without asking for more, and two
// workgroups a CU still fit.  Four lanes on 64 masses: up to 25 groups a block (the quadruped's 16 at most).
constexpr size_t kAdjBlockLds = 64 * 1024;

}  // namespace

hipError_t launch_step(const DeviceArrays& d, int cur, const StepParams& p, hipStream_t st) {
    return launch_step_io(d, d.x[cur], d.v[cur], d.x[cur ^ 1], d.v[cur ^ 1], nullptr, p, st, nullptr,
                          fused_actuation(d) ? 1 : 0, cur);
}

// Dynamic LDS of one step workgroup: positions, then (table and split modes) the parameter
// table and the workgroup's actuation factors, then (split mode) the spring factors.
hipError_t step_static_lds(size_t* bytes) {
    const void* ks[] = {(const void*)step_kernel<false, true, 4, kTable>, (const void*)step_kernel<true, true, 4, kTable>,
                        (const void*)step_persistent<false, true, 4, kTable>, (const void*)step_kernel<true, true, 4, kSplit>,
                        (const void*)step_persistent<true, false, 8, kSplit>,
                        (const void*)step_kernel<false, true, 4, kNarrow>,
                        (const void*)step_lanes_kernel<true, true, 4, false, true>,
                        (const void*)step_lanes_kernel<false, true, 2, true, false>,
                        (const void*)step_resident<false, true, 4, true, true>, (const void*)step_resident<true, true, 4, false, false>};
    *bytes = 0;
    for (const void* k : ks) {
        hipFuncAttributes at{};
        hipError_t e = hipFuncGetAttributes(&at, k);
        if (e != hipSuccess) return e;
        *bytes = std::max(*bytes, (size_t)at.sharedSizeBytes);
    }
    return hipSuccess;
}

size_t step_lds_bytes(const DeviceArrays& d) {
    size_t b = (size_t)d.lds_slots * sizeof(float4);
    if (d.packed || d.narrow)
        b = table_base(d.lds_slots) + (size_t)d.n_table * sizeof(float4) + (size_t)(d.max_local_groups + 1) * sizeof(float);
    if (d.sp_rec) b += (size_t)(d.max_sp + 1) * sizeof(float);
    return b;
}

// Dynamic LDS of a one-lane step launch: the staging above, and with stage_io room for the old
// velocities and the new state of the block's masses (a float4 and six floats each) that
// step_block passes through LDS in mass order.  (The several-lanes kernel keeps direct
// accesses: on the small systems it serves, the extra barriers cost more than the scattered
// lines.)
size_t step_launch_lds_bytes(const DeviceArrays& d) {
    if (!d.stage_io) return step_lds_bytes(d);
    return std::max(step_lds_bytes(d), (size_t)d.block * (sizeof(float4) + 6 * sizeof(float)));
}

bool fused_actuation(const DeviceArrays& d) { return d.grp != nullptr && (d.sp_rec || d.narrow || d.packed); }

hipError_t launch_step_io(const DeviceArrays& d, const float4* xin, const float* vin, float4* xout, float* vout,
                          float* vstar, const StepParams& p, hipStream_t st, const float* factor, int fuse,
                          int cur) {
    if (d.grid) {
        if (fuse) return hipErrorInvalidValue;
        GridArgs g{xin, vin, xout, vout, vstar, d.fext, d.grid_halo, d.grid_org, d.grid_k, d.grid_tab, (int)d.nblk,
                   d.grid_dim[0], d.grid_dim[1], d.grid_dim[2], {}, {}, {}};
        for (int q = 0; q < 3; ++q) {
            g.kin[q] = d.grid_kin[q];
            g.l0[q] = d.grid_l0[q];
            g.q[q] = (double)d.grid_l0[q] * (double)d.grid_l0[q];
        }
        const dim3 grid((unsigned)grid_for(d.nblk)), th(kGridThreads);
        if (p.exact) hipLaunchKernelGGL(step_grid_kernel<true>, grid, th, 0, st, g, p);
        else hipLaunchKernelGGL(step_grid_kernel<false>, grid, th, 0, st, g, p);
        return hipGetLastError();
    }
    const int mode = step_mode(d);
    if (fuse && !fused_actuation(d)) return hipErrorInvalidValue;
    StepArgs a{xin, vin, xout, vout, d.slice_ptr, d.nbr, d.kl, d.grp, d.halo_ptr, d.halo_idx,
               d.lane_mass, factor ? factor : d.factor, d.fext, vstar, d.packed, d.narrow, d.table, d.blk_groups, d.sp_rec, d.sp_grp,
               d.sp_ptr, (int)d.n, (int)d.nblk, (int)d.nslice, d.block, d.n_table, d.lds_slots, d.max_local_groups,
               d.narrow_tb, fuse, d.phase, d.amp, d.step_ctr + (cur & 1), d.step_ctr + ((cur & 1) ^ 1), d.act};
    const size_t lds = step_lds_bytes(d);
    if (d.lanes > 1 && (mode == kTable || mode == kNarrow)) {
        const bool act = d.grp != nullptr, ex = p.exact != 0, nar = mode == kNarrow && !act;
        const dim3 g((unsigned)grid_for(d.nblk)), th((unsigned)(d.block * d.lanes));
        auto go = [&](auto k) { hipLaunchKernelGGL(k, g, th, lds, st, a, p); };
#define CRONOS_GO_L(A, L, N, Y) (ex ? go(step_lanes_kernel<A, true, L, N, Y>) : go(step_lanes_kernel<A, false, L, N, Y>))
#define CRONOS_GO_LN(L, Y) (act ? CRONOS_GO_L(true, L, false, Y) : nar ? CRONOS_GO_L(false, L, true, Y) : CRONOS_GO_L(false, L, false, Y))
        const bool early = lanes_early(d);
        if (d.lanes == 2) early ? CRONOS_GO_LN(2, true) : CRONOS_GO_LN(2, false);
        else early ? CRONOS_GO_LN(4, true) : CRONOS_GO_LN(4, false);
#undef CRONOS_GO_LN
#undef CRONOS_GO_L
        return hipGetLastError();
    }
    if (mode == kExplicit && d.persistent_groups <= 0 && quads(d)) {
        const dim3 g((unsigned)grid_for(d.nblk)), th((unsigned)(4 * d.block));
        auto go = [&](auto k) { hipLaunchKernelGGL(k, g, th, lds, st, a, p); };
        if (d.grp) p.exact ? go(step_quads_kernel<true, true>) : go(step_quads_kernel<true, false>);
        else p.exact ? go(step_quads_kernel<false, true>) : go(step_quads_kernel<false, false>);
        return hipGetLastError();
    }
    const bool persistent = d.persistent_groups > 0;
    const dim3 grid(persistent ? (unsigned)d.persistent_groups : (unsigned)grid_for(d.nblk));
    const size_t lds1 = step_launch_lds_bytes(d);
    auto go = [&](auto normal, auto pers) {
        if (persistent) hipLaunchKernelGGL(pers, grid, dim3(d.block), lds1, st, a, p);
        else hipLaunchKernelGGL(normal, grid, dim3(d.block), lds1, st, a, p);
    };
#define CRONOS_GO(A, E, B, M) go(step_kernel<A, E, B, M>, step_persistent<A, E, B, M>)
// (16-bit entries exist for passive simulations only: the actuated expansion maps them to kTable,
// which it never meets there)
#define CRONOS_GO_M(A, E, B)                                                                         \
    (mode == kSplit    ? CRONOS_GO(A, E, B, kSplit)                                                  \
     : mode == kNarrow ? CRONOS_GO(A, E, B, (A ? kTable : kNarrow))                                  \
     : mode == kTable  ? CRONOS_GO(A, E, B, kTable)                                                  \
                       : CRONOS_GO(A, E, B, kExplicit))
    const bool act = d.grp != nullptr, ex = p.exact != 0;
    const int batch = step_batch(d, mode);
    if (d.stage_io && act && mode == kTable) {
#define CRONOS_GO_S(E, B) go(step_kernel<true, E, B, kTable, true>, step_persistent<true, E, B, kTable, true>)
        if (batch == 8) ex ? CRONOS_GO_S(true, 8) : CRONOS_GO_S(false, 8);
        else ex ? CRONOS_GO_S(true, 4) : CRONOS_GO_S(false, 4);
#undef CRONOS_GO_S
    } else if (batch == 8) {
        if (act) ex ? CRONOS_GO_M(true, true, 8) : CRONOS_GO_M(true, false, 8);
        else ex ? CRONOS_GO_M(false, true, 8) : CRONOS_GO_M(false, false, 8);
    } else if (batch == 2) {   // see step_batch
        if (mode == kSplit) ex ? CRONOS_GO(true, true, 2, kSplit) : CRONOS_GO(true, false, 2, kSplit);
        else ex ? CRONOS_GO(true, true, 2, kExplicit) : CRONOS_GO(true, false, 2, kExplicit);
    } else {
        if (act) ex ? CRONOS_GO_M(true, true, 4) : CRONOS_GO_M(true, false, 4);
        else ex ? CRONOS_GO_M(false, true, 4) : CRONOS_GO_M(false, false, 4);
    }
#undef CRONOS_GO_M
#undef CRONOS_GO
    return hipGetLastError();
}

hipError_t launch_resident(const DeviceArrays& d, int cur, const StepParams& p, float dtv0, unsigned long long cycles,
                           int steps, hipStream_t st) {
    StepArgs a{d.x[cur], d.v[cur], d.x[cur ^ 1], d.v[cur ^ 1], d.slice_ptr, d.nbr, d.kl, d.grp, d.halo_ptr, d.halo_idx,
               d.lane_mass, d.factor, d.fext, nullptr, d.packed, d.narrow, d.table, d.blk_groups, d.sp_rec, d.sp_grp,
               d.sp_ptr, (int)d.n, (int)d.nblk, (int)d.nslice, d.block, d.n_table, d.lds_slots, d.max_local_groups,
               d.narrow_tb, 0, d.phase, d.amp, d.step_ctr + (cur & 1), d.step_ctr + ((cur & 1) ^ 1), d.act};
    ResidentArgs r{d.phase, d.amp, cycles, d.step_ctr + (cur & 1), d.step_ctr + ((cur & 1) ^ 1), steps, dtv0,
                   d.resident_staged};
    const size_t lds = step_lds_bytes(d) + (size_t)d.resident_staged * sizeof(uint32_t);
    const bool act = d.grp != nullptr, ex = p.exact != 0;
    auto go = [&](auto k) { hipLaunchKernelGGL(k, dim3(1), dim3(d.block), lds, st, a, p, r); };
    const bool ahead = d.block > 512;   // see step_resident
#define CRONOS_GO_R(A, E, S) (ahead ? go(step_resident<A, E, 4, S, true>) : go(step_resident<A, E, 4, S, false>))
    if (d.resident_staged) {
        if (act) ex ? CRONOS_GO_R(true, true, true) : CRONOS_GO_R(true, false, true);
        else ex ? CRONOS_GO_R(false, true, true) : CRONOS_GO_R(false, false, true);
    } else {
        if (act) ex ? CRONOS_GO_R(true, true, false) : CRONOS_GO_R(true, false, false);
        else ex ? CRONOS_GO_R(false, true, false) : CRONOS_GO_R(false, false, false);
    }
#undef CRONOS_GO_R
    return hipGetLastError();
}

hipError_t persistent_grid(const DeviceArrays& d, int exact, int* grid) {
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    // the very kernel that will run: a grid of more workgroups than the device holds at once takes two rounds
    const void* k = nullptr;
    const int mode = step_mode(d), batch = step_batch(d, mode);
    const bool act = d.grp != nullptr;
    auto is = [&](const void* kernel) { k = kernel; };
#define CRONOS_K(A, E, B, M) (const void*)step_persistent<A, E, B, M>
#define CRONOS_K_M(A, E, B)                                                                                       \
    is(mode == kSplit ? CRONOS_K(A, E, B, kSplit) : mode == kNarrow ? CRONOS_K(A, E, B, (A ? kTable : kNarrow))   \
       : mode == kTable ? CRONOS_K(A, E, B, kTable) : CRONOS_K(A, E, B, kExplicit))
#define CRONOS_K_E(A, B) (exact ? CRONOS_K_M(A, true, B) : CRONOS_K_M(A, false, B))
    if (batch == 2) {   // actuated split and explicit forms only
        if (mode == kSplit) is(exact ? CRONOS_K(true, true, 2, kSplit) : CRONOS_K(true, false, 2, kSplit));
        else is(exact ? CRONOS_K(true, true, 2, kExplicit) : CRONOS_K(true, false, 2, kExplicit));
    } else if (batch == 8) {
        act ? CRONOS_K_E(true, 8) : CRONOS_K_E(false, 8);
    } else {
        act ? CRONOS_K_E(true, 4) : CRONOS_K_E(false, 4);
    }
#undef CRONOS_K_E
#undef CRONOS_K_M
#undef CRONOS_K
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, d.block, step_launch_lds_bytes(d));
    if (e != hipSuccess) return e;
    int g = std::max(1, per_cu) * cus;
    g = (g + 7) / 8 * 8;
    *grid = (int)std::min<int64_t>(g, grid_for(d.nblk));
    return hipSuccess;
}

hipError_t launch_actuation(const DeviceArrays& d, int advance, hipStream_t st,
                            long long n_explicit, float* out, int cur) {
    const unsigned grid = (unsigned)((d.n_factor + 1 + 255) / 256);
    hipLaunchKernelGGL(actuation_kernel, dim3(grid), dim3(256), 0, st, d.phase, d.amp, d.act, d.step_ctr + (cur & 1),
                       d.step_ctr + ((cur & 1) ^ 1), out ? out : d.factor, d.n_factor, n_explicit >= 0 ? 0 : advance,
                       n_explicit);
    return hipGetLastError();
}

hipError_t launch_forces(const DeviceArrays& d, int cur, const StepParams& p, hipStream_t st) {
    const int nslice = (int)d.nslice;
    const size_t lds = (size_t)d.lds_slots * sizeof(float4);
    if (d.grp)
        hipLaunchKernelGGL(forces_kernel<true>, dim3(grid_for(d.nblk)), dim3(d.block), lds, st, d.x[cur], d.mass,
                           d.slice_ptr, d.nbr, d.kl, d.grp, d.halo_ptr, d.halo_idx, d.lane_mass, d.factor, d.fext,
                           d.fout, (int)d.n, (int)d.nblk, nslice, d.block, p);
    else
        hipLaunchKernelGGL(forces_kernel<false>, dim3(grid_for(d.nblk)), dim3(d.block), lds, st, d.x[cur], d.mass,
                           d.slice_ptr, d.nbr, d.kl, d.grp, d.halo_ptr, d.halo_idx, d.lane_mass, d.factor, d.fext,
                           d.fout, (int)d.n, (int)d.nblk, nslice, d.block, p);
    return hipGetLastError();
}

hipError_t launch_diagnostics(const DeviceArrays& d, int cur, const StepParams& p, double* out, hipStream_t st) {
    const int nslice = (int)d.nslice;
    const size_t lds = (size_t)d.lds_slots * sizeof(float4);
    if (d.grp)
        hipLaunchKernelGGL(diag_chunk_kernel<true>, dim3(d.n_chunks), dim3(d.block), lds, st, d.x[cur], d.v[cur],
                           d.mass, d.slice_ptr, d.nbr, d.kl, d.grp, d.halo_ptr, d.halo_idx, d.lane_mass, d.factor,
                           d.chunks, d.chunk_part, (int)d.n, nslice, d.block, p);
    else
        hipLaunchKernelGGL(diag_chunk_kernel<false>, dim3(d.n_chunks), dim3(d.block), lds, st, d.x[cur], d.v[cur],
                           d.mass, d.slice_ptr, d.nbr, d.kl, d.grp, d.halo_ptr, d.halo_idx, d.lane_mass, d.factor,
                           d.chunks, d.chunk_part, (int)d.n, nslice, d.block, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(diag_body_kernel, dim3((unsigned)d.nb), dim3(64), 0, st, d.chunk_part, d.body_chunk, out);
    return hipGetLastError();
}

hipError_t launch_adj_local(const DeviceArrays& d, const float4* x, const float* vstar, const float* xb1,
                            const float* vb1, float4* w, float* vb0, float* xbl, const StepParams& p, hipStream_t st) {
    hipLaunchKernelGGL(adj_local_kernel, dim3((unsigned)((d.n + 255) / 256)), dim3(256), 0, st, x, vstar, xb1, vb1, w,
                       vb0, xbl, (int)d.n, p);
    return hipGetLastError();
}

hipError_t launch_actuation_steps(const DeviceArrays& d, unsigned long long cycles, long long n0, int steps,
                                  float* out, long long stride, hipStream_t st) {
    const unsigned grid = (unsigned)((d.n_factor + 1 + 255) / 256);
    for (int k0 = 0; k0 < steps; k0 += 65535) {   // at most 65535 rows per launch (grid y)
        const int rows = std::min(steps - k0, 65535);
        hipLaunchKernelGGL(actuation_steps_kernel, dim3(grid, (unsigned)rows), dim3(256), 0, st, d.phase, d.amp, cycles,
                           n0 + k0, out + (size_t)k0 * (size_t)stride, d.n_factor, stride);
    }
    return hipGetLastError();
}

namespace {

// LDS of a reverse step whose workgroups sum up to `groups` groups each (0: none of its own), a row
// more than that for the springs that count towards none of them.
size_t adj_lds_bytes(const DeviceArrays& d, int groups) {
    const size_t threads = (size_t)d.block * (d.lanes == 2 || d.lanes == 4 ? d.lanes : 1);
    return 2 * (size_t)d.lds_slots * sizeof(float4) + (groups ? (size_t)(groups + 1) * ((threads + 16) * sizeof(double) + sizeof(float)) : 0);
}

}  // namespace

// Sums per workgroup pay where they save more than they cost.  They save a read and a write of 16 bytes per
// entry, which is the more the less of them the caches hold; they cost each thread two LDS operations per group
// of the workgroup's range, and LDS that other workgroups could use.  Per entry / per workgroup, us a
// reversed step with the step recomputed beside it: 4 lanes on 64 masses, 16 groups, 26 rows a mass, 1,000 masses
// 14.5 / 13.6, 12,000 16.4 / 14.4, 50,000 28.9 / 21.8; 14 rows 12.0 / 12.5, 13.3 / 12.7, 21.9 / 19.2; 4
// rows 10.2 / 11.3, 10.9 / 11.2, 15.3 / 14.1; 24 groups, 14 rows 12.6 / 13.7, 13.2 / 13.6, 20.8 / 21.7; one lane,
// 40 groups in 64-mass workgroups, 8 rows 13.0 / 17.3, 14.8 / 18.0, 17.4 / 19.7.
// (No group at all: the passive form, which sums nothing.)
bool adj_block_sums(const DeviceArrays& d, int max_groups) {
    if (max_groups == 0) return true;
    if (adj_lds_bytes(d, max_groups) > kAdjBlockLds) return false;
    const float groups = (float)max_groups, threads = (float)(d.block * d.lanes);
    if (d.n < 8192) return d.mean_rows >= 20.0f && groups <= d.mean_rows && 16.0f * groups <= 3.0f * threads;
    return groups <= (d.n < 32768 ? 1.0f : 2.0f) * d.mean_rows;
}

hipError_t launch_adj_gather(const DeviceArrays& d, const float4* x, const float4* w, const float* xbl, float* xb0,
                             double2* sens, const int4* range, int max_groups, double cos_t, double sin_t, hipStream_t st,
                             const float* factor, const StepParams& p, const AdjNext& next) {
    if (!factor) factor = d.factor;
    // kAdjEntrySums: the factor table goes to LDS when small (kAdjStagedFactors entries at most)
    const int stage = d.grp && !range && d.n_factor + 1 <= kAdjStagedFactors ? 1 : 0;
    const size_t lds = range ? adj_lds_bytes(d, max_groups)
                             : adj_lds_bytes(d, 0) + (stage ? (size_t)(d.n_factor + 1) * sizeof(float) : 0);
    const int lanes = d.lanes == 2 || d.lanes == 4 ? d.lanes : 1;
    const dim3 g(grid_for(d.nblk)), th((unsigned)(d.block * lanes));
    const AdjArgs a{x, w, xbl, xb0, d.slice_ptr, d.nbr, d.kl, d.grp, d.halo_ptr, d.halo_idx, d.lane_mass, factor, sens, range,
                    cos_t, sin_t, d.n_factor, (int)d.n, (int)d.nblk, (int)d.nslice, d.block, d.lds_slots, max_groups, stage};
    auto go = [&](auto one, auto two, auto four) {
        const auto k = lanes == 4 ? four : lanes == 2 ? two : one;
        hipLaunchKernelGGL(k, g, th, lds, st, a, p, next);
    };
#define CRONOS_ADJ(M) go(adj_gather_kernel<M>, adj_gather_lanes_kernel<M, 2>, adj_gather_lanes_kernel<M, 4>)
    // a body with groups of which no spring is a member has nothing to sum, and factors of 1 only
    if (!d.grp || (range && max_groups == 0)) CRONOS_ADJ(kAdjPassive);
    else if (range) CRONOS_ADJ(kAdjBlockSums);
    else CRONOS_ADJ(kAdjEntrySums);
#undef CRONOS_ADJ
    return hipGetLastError();
}

namespace {

// State between the device's mass order and the caller's, in pinned host memory that the kernels
// read and write themselves (a copy after the kernel would be another launch and another pass).  The
// permutation is done here, where scattered accesses are cheap, so that the host only converts
// between FP32 and FP64 along its arrays: 640,000 masses read in 1.6 ms against 4.0 (the host's own
// scatter), set in 1.7 ms against 5.9.
// A workgroup takes 256 masses of the caller's order; its part of the host array is moved 16 bytes
// a lane, through LDS.
constexpr int kIoMasses = 256;

__device__ __forceinline__ void io_out(const float* __restrict__ sh, float* __restrict__ host, int floats) {
    for (int q = (int)threadIdx.x; q < 3 * kIoMasses / 4; q += kIoMasses) {
        if (4 * q + 4 <= floats)
            reinterpret_cast<float4*>(host)[q] = make_float4(sh[4 * q], sh[4 * q + 1], sh[4 * q + 2], sh[4 * q + 3]);
        else
            for (int c = 4 * q; c < floats; ++c) host[c] = sh[c];
    }
}

__device__ __forceinline__ void io_in(float* __restrict__ sh, const float* __restrict__ host, int floats) {
    for (int q = (int)threadIdx.x; q < 3 * kIoMasses / 4; q += kIoMasses) {
        if (4 * q + 4 <= floats) {
            const float4 w = reinterpret_cast<const float4*>(host)[q];
            sh[4 * q] = w.x;
            sh[4 * q + 1] = w.y;
            sh[4 * q + 2] = w.z;
            sh[4 * q + 3] = w.w;
        } else {
            for (int c = 4 * q; c < floats; ++c) sh[c] = host[c];
        }
    }
}

// Masses [o0, o0 + count) of the caller's order: positions x and a 3-vector array v (either may be null).
__global__ void __launch_bounds__(kIoMasses)
unpack_kernel(const float4* __restrict__ x, const float* __restrict__ v, const int32_t* __restrict__ inv,
              float* __restrict__ host_x, float* __restrict__ host_v, int o0, int count) {
    __shared__ float sx[3 * kIoMasses], sv[3 * kIoMasses];
    const int t = (int)threadIdx.x, first = (int)blockIdx.x * kIoMasses, mine = min(kIoMasses, count - first);
    if (t < mine) {
        const long i = inv[o0 + first + t];
        if (x) {
            const float4 p = x[i];
            sx[3 * t] = p.x;
            sx[3 * t + 1] = p.y;
            sx[3 * t + 2] = p.z;
        }
        if (v)
            for (int c = 0; c < 3; ++c) sv[3 * t + c] = v[3 * i + c];
    }
    __syncthreads();
    if (x) io_out(sx, host_x + 3 * (long)first, 3 * mine);
    if (v) io_out(sv, host_v + 3 * (long)first, 3 * mine);
}

// The other way, into xo and vo; 1/m of each mass from `now`, and v = 0 for fixed masses.
__global__ void __launch_bounds__(kIoMasses)
pack_kernel(const float* __restrict__ host_x, const float* __restrict__ host_v, const int32_t* __restrict__ inv,
            const float4* __restrict__ now, float4* __restrict__ xo, float* __restrict__ vo, int o0, int count) {
    __shared__ float sx[3 * kIoMasses], sv[3 * kIoMasses];
    const int t = (int)threadIdx.x, first = (int)blockIdx.x * kIoMasses, mine = min(kIoMasses, count - first);
    if (xo) io_in(sx, host_x + 3 * (long)first, 3 * mine);
    if (vo) io_in(sv, host_v + 3 * (long)first, 3 * mine);
    __syncthreads();
    if (t >= mine) return;
    const long i = inv[o0 + first + t];
    const float w = now[i].w;
    if (xo) xo[i] = make_float4(sx[3 * t], sx[3 * t + 1], sx[3 * t + 2], w);
    if (vo)
        for (int c = 0; c < 3; ++c) vo[3 * i + c] = w == 0.0f ? 0.0f : sv[3 * t + c];
}

// Makes a packed state the current one (xs or vs null: that part is kept) at step `step`.
__global__ void __launch_bounds__(256)
commit_state_kernel(const float4* __restrict__ xs, const float* __restrict__ vs, float4* __restrict__ x,
                    float* __restrict__ v, int n, long long* __restrict__ step_ctr, long long step) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i == 0) *step_ctr = step;
    if (i >= n) return;
    if (xs) x[i] = xs[i];
    if (vs)
        for (int c = 0; c < 3; ++c) v[3 * (long)i + c] = vs[3 * (long)i + c];
}

}  // namespace

hipError_t launch_unpack(const float4* x, const float* v, const int32_t* inv, float* host_x, float* host_v, int o0,
                         int count, hipStream_t st) {
    hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)((count + kIoMasses - 1) / kIoMasses)), dim3(kIoMasses), 0, st, x, v,
                       inv, host_x, host_v, o0, count);
    return hipGetLastError();
}

hipError_t launch_pack(const float* host_x, const float* host_v, const int32_t* inv, const float4* now, float4* xo,
                       float* vo, int o0, int count, hipStream_t st) {
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((count + kIoMasses - 1) / kIoMasses)), dim3(kIoMasses), 0, st, host_x,
                       host_v, inv, now, xo, vo, o0, count);
    return hipGetLastError();
}

hipError_t launch_commit_state(const DeviceArrays& d, int cur, bool x, bool v, long long step, hipStream_t st) {
    hipLaunchKernelGGL(commit_state_kernel, dim3((unsigned)((d.n + 255) / 256)), dim3(256), 0, st,
                       x ? d.x[cur ^ 1] : nullptr, v ? d.v[cur ^ 1] : nullptr, d.x[cur], d.v[cur], (int)d.n,
                       d.step_ctr + (cur & 1), step);
    return hipGetLastError();
}

namespace {

// One workgroup per actuation group: its sums (one per entry or per workgroup), each thread over a
// strided part of the group's list in order, then the fixed-order workgroup tree.
__global__ void __launch_bounds__(256) adj_group_sums_kernel(const double2* __restrict__ sens,
                                                             const int32_t* __restrict__ grp_ptr,
                                                             const int32_t* __restrict__ grp_sums,
                                                             double2* __restrict__ gsum) {
    __shared__ double2 red[256];
    const int g = blockIdx.x, t = threadIdx.x;
    double2 s = make_double2(0.0, 0.0);
    for (int q = grp_ptr[g] + t; q < grp_ptr[g + 1]; q += 256) {
        const double2 v = sens[grp_sums[q]];
        s.x += v.x;
        s.y += v.y;
    }
    red[t] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) {
            red[t].x += red[t + h].x;
            red[t].y += red[t + h].y;
        }
        __syncthreads();
    }
    if (t == 0) gsum[g] = red[0];
}

}  // namespace

hipError_t launch_adj_group_sums(const double2* sens, const int32_t* grp_ptr, const int32_t* grp_sums, int n_groups,
                                 double2* gsum, hipStream_t st) {
    if (n_groups < 1) return hipSuccess;
    hipLaunchKernelGGL(adj_group_sums_kernel, dim3(n_groups), dim3(256), 0, st, sens, grp_ptr, grp_sums, gsum);
    return hipGetLastError();
}

}  // namespace cronos
