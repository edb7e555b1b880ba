// Surrogate network on gfx950: a 4-layer perceptron (3 exact-erf GELU hidden layers, linear
// output) whose products run on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16) with FP32
// accumulation; weights are kept as an FP32 master copy and two BF16 shadows; Adam in FP32.
//
// Every product is C[M x N] = A B^T with both operands stored K-contiguous (A: M rows of K,
// B: N rows of K), so each operand tile arrives with 16-byte vector loads along K.  To keep it
// that way the network stores, beside each row-major activation it produces, its transpose
// (written by the producing product's epilogue), and keeps both W and W^T as BF16 shadows:
//   forward      Z_l = H_{l-1} W_l        A = H_{l-1} (rows x in),   B = W_l^T (out x in)
//   input grad   dH  = dZ_l W_l^T         A = dZ_l (rows x out),     B = W_l   (in x out)
//   weight grad  [dW_l; db_l] = [H^T; 1] dZ_l   A = [H_{l-1}^T; ones] (in+1 x rows),
//                                               B = dZ_l^T (out x rows)
// The row of ones appended to each transposed input makes the bias gradient (a column sum
// of dZ) the last row of the weight-gradient product, which lands exactly where the bias
// follows the weight in the parameter vector.  Widths are padded to multiples of 32 with zero
// weights, so padded activations are exactly zero.
//
// Tiling: a workgroup of 8 wavefronts computes a 64 x 64 tile of C (128 x 128 for forward products of
// many rows), each wavefront an eighth of it in MFMA tiles of 16 x 16, stepping K by 64 (or 32)
// through a ring of four LDS stages.  A minibatch's product is a few hundred
// tiles, one workgroup per CU or two, so nothing but its own wavefronts hides a latency: eight of them,
// and the operands of three K-steps on their way at once, straight from memory into an LDS ring
// (no registers, no store; one barrier per step).  1024 x 768 x 768 with GELU, its slope and
// the transposed output: 11.5 -> 8.2 us; the paired backward products 16.2 -> 10.4 us (four
// wavefronts, one step of 128 ahead in registers, both GELU and slope by erf per element).  The
// weight gradients (K = the minibatch rows) split K into chunks of 512 rows computed by separate
// workgroups into FP32 partials, laid out like the parameters, that Adam adds in a fixed
// order (or one more kernel, when the gradient itself is asked for).  Every element of C sums K in
// ascending steps of 32, whatever the tile and the K-step, so those do not change a bit of it.
// Operand layouts of the 16x16x32 BF16 MFMA: lane l supplies A[l % 16][8 (l / 16) + j] and
// B[8 (l / 16) + j][l % 16], j = 0..7, and receives C[4 (l / 16) + r][l % 16], r = 0..3.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "common.h"

namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;           // workgroup tile (rows and columns); 128 where launch_forward takes it
constexpr int kThreads = 512;       // of a product's workgroup: 8 wavefronts, 2 across the tile's rows, 4 across its columns
constexpr int kStages = 4;          // K-steps of operands held in LDS, three of them in flight
constexpr int kWidthPad = 32;       // widths are padded to multiples of this (the MFMA's K)
constexpr int kSplitRows = 512;     // K chunk of the weight-gradient products

enum Epilogue { kFwdGelu = 0, kLinear = 1, kBwdGelu = 2, kPartial = 3 };

struct GemmArgs {
    const bf16* A;
    long lda;             // A(m, k) = A[m * lda + k], m < M
    const bf16* B;
    long ldb;             // B(n, k) = B[n * ldb + k], n < N
    int M, N, K;          // K: a multiple of the K-step; lda, ldb: multiples of 8
    int k_chunk;          // K range of workgroup z: [z k_chunk, (z + 1) k_chunk)
    int n_real;           // columns below n_real get the bias, the transposed and FP32 outputs
    const float* bias;    // [n_real] (forward epilogues)
    float* Cf;            // FP32 output: Cf[m * ldcf + n] (+ z * part_stride for partials); the forward's are
                          // the activation's slopes gelu'(Z), for the backward (null: left out, and with
                          // them the transposed output)
    long ldcf, part_stride;
    bf16* Cb;             // BF16 row-major output: Cb[m * ldcb + n], n < N
    long ldcb;
    bf16* Ct;             // BF16 transposed output: Ct[n * ldct + m], n < n_real
    long ldct;
    const float* S;       // the activation's slopes S[m * lds + n] (backward GELU)
    long lds;
    int nbx, nby, tiles;  // column tiles, row tiles and their product with the K-splits
    // linear output with the loss (T non-null): dY = 2 (Y - T) / (rows n_real) as BF16, row-major
    // dY[m * lddy + n] for n < N (zero beyond n_real and below M beyond `rows`) and transposed
    // dYt[n * lddyt + m] for n < n_real; the sum of squares of Y - T per tile in loss_part
    const float* T;       // targets T[m * n_real + n], m < rows
    bf16* dY;
    long lddy;
    bf16* dYt;
    long lddyt;
    double* loss_part;
    int rows;
};

constexpr float kRsqrt2 = 0.70710678118654752f;

// GELU and its slope at z, given e = erf(z / sqrt 2).
__device__ __forceinline__ float gelu(float z, float e) { return 0.5f * z * (1.0f + e); }

__device__ __forceinline__ float gelu_grad(float z, float e) {
    return 0.5f * (1.0f + e) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// e[i] = erff(x[i]) for N values per lane.  erff takes a short polynomial below 1 and a much longer way
// above; of 64 normally distributed pre-activations a few always lie above, so a wavefront that
// evaluates value after value takes both ways every time (155 instructions per GELU and slope,
// half of a product's time).  Here the values from 1 on (a sixth) are queued in LDS without gaps
// and evaluated 64 at a time.  The results are erff's own either way.  queue: 64 (N + 1) floats of this
// wavefront's, used by no other.
template <int N>
__device__ __forceinline__ void erf_values(const float (&x)[N], float (&e)[N], float* queue) {
    // a value's place in the queue; one evaluated here writes to and reads from the lane's spare place
    uint32_t place[N];
    bool wide[N];
    const uint32_t spare = 64 * N + (threadIdx.x & 63);
    int queued = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        wide[i] = !(fabsf(x[i]) < 1.0f);
        const unsigned long long who = __builtin_amdgcn_ballot_w64(wide[i]);
        const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)who, (uint32_t)queued));
        place[i] = wide[i] ? at : spare;
        queue[place[i]] = x[i];
        queued += __builtin_popcountll(who);
        // no branch here either: the values' polynomials overlap
        float near = wide[i] ? 0.0f : x[i];
        asm("" : "+v"(near));   // (the compiler does not see that it is below 1 through the selection)
        __builtin_assume(__builtin_fabsf(near) < 1.0f);
        e[i] = erff(near);
    }
    // one wavefront's LDS accesses execute in order; the compiler is held to it as well
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    for (int q = (int)(threadIdx.x & 63); q < queued; q += 64) queue[q] = erff(queue[q]);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float far = queue[place[i]];
        e[i] = wide[i] ? far : e[i];
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t pack2(bf16 lo, bf16 hi) {
    return (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
}

// Elements of one operand's LDS: a ring of kStages K-steps of T rows of BK; later, for the GELU epilogues,
// the tile's FP32 sums at a pitch of T + 4 (A's), its transposed BF16 outputs at a pitch of T + 8 and four
// wavefronts' queues of erf_values (B's).
constexpr int kErfPieces = 2;
template <int BK, int T>
constexpr int kLdsElems = std::max({kStages * T * BK, 2 * T * (T + 4), T * (T + 8) + kThreads * (4 * kErfPieces + 1) * 2});

// 16 bytes per lane from global memory (byte offset `from` of `src`) straight into LDS, at byte address
// lds + AT + 16 * lane; src and lds are uniform over the wavefront.  Counted by vmcnt like any
// load, in order; no register is written.
template <int AT>
__device__ __forceinline__ void load_to_lds(const bf16* src, uint32_t from, uint32_t lds) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds), "v"(from), "s"(src), "n"(AT)
                 : "m0", "scc", "memory");
}

// Waits until at most `newer` of this wavefront's later loads are still on their way.
template <int NEWER>
__device__ __forceinline__ void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NEWER) : "memory");
}

// One workgroup's T x T tile (column tile bx, row tile by, K-split bz) of the product g, staged
// through As / Bs (kLdsElems each, at least).
template <int EPI, int BK, int T>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, int bx, int by, int bz, bf16* As,
                                          bf16* Bs) {
    constexpr int CPR = BK / 8;               // 16-byte chunks per tile row
    constexpr int CHUNKS = T * CPR;           // 16-byte pieces of an operand's K-step
    // loads per thread per K-step: of both operands, or (half a workgroup's worth each) of one
    constexpr bool SHARED = CHUNKS < kThreads;
    constexpr int PER = SHARED ? 1 : CHUNKS / kThreads, LOADS = SHARED ? 1 : 2 * PER;
    constexpr int BUF = T * BK;               // elements of one stage
    constexpr int FM = T / 32, FN = T / 64;   // MFMA tiles of a wavefront along the rows and the columns
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int m0 = by * T, n0 = bx * T;
    const int kbeg = bz * g.k_chunk;
    const int kend = min(g.K, kbeg + g.k_chunk);
    const int nk = (kend - kbeg) / BK;
    const int wm = (wave >> 2) * (T / 2), wn = (wave & 3) * (T / 4);
    // A direct load writes a wavefront's 64 chunks one after the other, so rows cannot be padded; row
    // r's chunk c lies in place c ^ turn(r) instead, and the 16 rows that the MFMA operand reads
    // take together (the same chunk of each) fall into different banks.
    auto turn = [](int row) { return (row / (16 / CPR)) & (CPR - 1); };

    // rows past the operand's last repeat it: they reach only rows and columns of C that are not stored
    const bool does_a = !SHARED || wave < kThreads / 128, does_b = !SHARED || !does_a;
    const int t0 = SHARED ? t & (kThreads / 2 - 1) : t;
    static_assert(!SHARED || CHUNKS == kThreads / 2, "an operand's K-step is half a workgroup's loads or whole ones");
    uint32_t oa[PER], ob[PER];   // byte offsets from the tile's first element
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = t0 + kThreads * i, row = c / CPR, kc = ((c % CPR) ^ turn(row)) * 8;
        oa[i] = (uint32_t)(min(row, g.M - 1 - m0) * g.lda + kc) * 2u;
        ob[i] = (uint32_t)(min(row, g.N - 1 - n0) * g.ldb + kc) * 2u;
    }
    const bf16* const ga = g.A + (long)m0 * g.lda + kbeg;
    const bf16* const gb = g.B + (long)n0 * g.ldb + kbeg;
    const uint32_t la = __builtin_amdgcn_readfirstlane(
        (uint32_t)(size_t)(__attribute__((address_space(3))) bf16*)As + (uint32_t)((t0 >> 6) * 1024));
    const uint32_t lb = __builtin_amdgcn_readfirstlane(
        (uint32_t)(size_t)(__attribute__((address_space(3))) bf16*)Bs + (uint32_t)((t0 >> 6) * 1024));
    auto gload = [&](auto stage, int it) {
        constexpr int off = decltype(stage)::value * BUF * 2, more = kThreads * 16;
        const bf16 *sa = ga + it * BK, *sb = gb + it * BK;
        if (does_a) load_to_lds<off>(sa, oa[0], la);
        if (does_b) load_to_lds<off>(sb, ob[0], lb);
        if constexpr (PER == 2) {
            load_to_lds<off + more>(sa, oa[1], la);
            load_to_lds<off + more>(sb, ob[1], lb);
        }
    };
    static_assert(PER <= 2, "loads of a K-step");

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int r16 = lane & 15, k8 = lane >> 4;
    // what the epilogue reads beside the sums, loaded before the K-loop, which hides its latency: the
    // targets of a linear output with the loss (in the MFMA's output layout); for the GELU epilogues,
    // which work on four adjacent columns of a row at a time, the bias or the activation's slopes
    constexpr int Q4 = T / 4, ROWS = kThreads / Q4, PASSES = T / ROWS;
    const int qrow = t / Q4, qcol = t % Q4 * 4;   // this thread's first piece; further ones ROWS rows on
    float side[FM][FN][4] = {};
    f32x4 bias4 = f32x4{0.f, 0.f, 0.f, 0.f}, slope4[EPI == kBwdGelu ? PASSES : 1];
    if (EPI == kLinear && g.T) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int mb = m0 + wm + i * 16 + (lane >> 4) * 4, n = n0 + wn + j * 16 + (lane & 15);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (n < g.n_real && mb + r < g.rows) side[i][j][r] = g.T[(long)(mb + r) * g.n_real + n];
            }
    }
    if (EPI == kFwdGelu) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (n0 + qcol + c < g.n_real) bias4[c] = g.bias[n0 + qcol + c];
    }
    if constexpr (EPI == kBwdGelu) {
#pragma unroll
        for (int q = 0; q < PASSES; ++q) {
            const int m = min(m0 + qrow + q * ROWS, g.M - 1), n = min(n0 + qcol, g.N - 4);   // outside: unused
            slope4[q] = *reinterpret_cast<const f32x4*>(g.S + (long)m * g.lds + n);
        }
    }

    // operand places in a stage: row r of 16 i + r16 turns alike for every i
    const int ra = (wm + r16) * BK, rb = (wn + r16) * BK, tn = turn(r16);
    static_assert(BK * 16 % 128 == 0, "rows 16 apart turn alike");
    auto step = [&](auto stage, int it) {
        constexpr int u = decltype(stage)::value;
        // this wavefront's part of step `it` has arrived once only the newer steps' loads remain ...
        const int newer = min(nk - 1 - it, kStages - 2);
        if (newer == 2) wait_loads<2 * LOADS>();
        else if (newer == 1) wait_loads<LOADS>();
        else wait_loads<0>();
        // ... and the others' after the barrier, which also frees the stage of step it - 1
        __syncthreads();
        if (it + kStages - 1 < nk) gload(std::integral_constant<int, (u + kStages - 1) % kStages>{}, it + kStages - 1);
#pragma unroll
        for (int ks = 0; ks < CPR; ks += 4) {
            bf16x8 a[FM], b[FN];
            const int kc = ((ks + k8) ^ tn) * 8;
#pragma unroll
            for (int i = 0; i < FM; ++i)
                a[i] = *reinterpret_cast<const bf16x8*>(As + ra + kc + (u * BUF + i * 16 * BK));
#pragma unroll
            for (int j = 0; j < FN; ++j)
                b[j] = *reinterpret_cast<const bf16x8*>(Bs + rb + kc + (u * BUF + j * 16 * BK));
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    using S3 = std::integral_constant<int, 3>;
    if (0 < nk) gload(S0{}, 0);
    if (1 < nk) gload(S1{}, 1);
    if (2 < nk) gload(S2{}, 2);
    for (int it = 0; it < nk; it += kStages) {
        step(S0{}, it);
        if (it + 1 < nk) step(S1{}, it + 1);
        if (it + 2 < nk) step(S2{}, it + 2);
        if (it + 3 < nk) step(S3{}, it + 3);
    }
    static_assert(kStages == 4, "the waits and stages above are of a ring of four");
    __syncthreads();   // the buffers are free

    if constexpr (EPI == kFwdGelu || EPI == kBwdGelu) {
        // The sums go through LDS, so that a thread has four adjacent columns of a row: every output
        // leaves in 8- or 16-byte pieces of rows (the transposed ones through LDS once more), and the
        // activation's code is a short loop (fully unrolled over the MFMA's output layout it was 1,900
        // instructions executed once: half of the product's time).  M is a multiple of 64, N of 32 (padded
        // minibatch rows and widths).
        constexpr int LDC = T + 4, LDT = T + 8;
        float* const c32 = reinterpret_cast<float*>(As);
        float* const queue = reinterpret_cast<float*>(Bs + T * LDT) + wave * (64 * (4 * kErfPieces + 1));
        const bool transposed = EPI == kBwdGelu || g.Cf;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    c32[(wm + i * 16 + (lane >> 4) * 4 + r) * LDC + wn + j * 16 + r16] = acc[i][j][r];
        __syncthreads();
        auto put = [&](int q, const bf16 (&h)[4]) {   // piece q's outputs
            const int row = qrow + q * ROWS, m = m0 + row, n = n0 + qcol;
            if (m < g.M && n < g.N)
                *reinterpret_cast<uint2*>(g.Cb + (long)m * g.ldcb + n) = uint2{pack2(h[0], h[1]), pack2(h[2], h[3])};
            if (transposed) {
#pragma unroll
                for (int c = 0; c < 4; ++c) Bs[(qcol + c) * LDT + row] = h[c];
            }
        };
        if constexpr (EPI == kBwdGelu) {
#pragma unroll
            for (int q = 0; q < PASSES; ++q) {
                const f32x4 sum = *reinterpret_cast<const f32x4*>(c32 + (qrow + q * ROWS) * LDC + qcol);
                bf16 h[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) h[c] = (bf16)(sum[c] * slope4[q][c]);
                put(q, h);
            }
        } else {
            constexpr int G = kErfPieces;   // pieces whose values go through erf_values together
#pragma unroll 1
            for (int q0 = 0; q0 < PASSES; q0 += G) {
                float z[4 * G], x[4 * G], e[4 * G];
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    const f32x4 sum = *reinterpret_cast<const f32x4*>(c32 + (qrow + (q0 + q) * ROWS) * LDC + qcol);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        z[4 * q + c] = sum[c] + bias4[c];
                        x[4 * q + c] = z[4 * q + c] * kRsqrt2;
                    }
                }
                erf_values(x, e, queue);
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    bf16 h[4];
                    f32x4 s;
#pragma unroll
                    for (int c = 0; c < 4; ++c) h[c] = (bf16)gelu(z[4 * q + c], e[4 * q + c]);
                    put(q0 + q, h);
                    const int m = m0 + qrow + (q0 + q) * ROWS, n = n0 + qcol;
                    if (!g.Cf) continue;
#pragma unroll
                    for (int c = 0; c < 4; ++c) s[c] = gelu_grad(z[4 * q + c], e[4 * q + c]);
                    if (m < g.M && n < g.N) *reinterpret_cast<f32x4*>(g.Cf + (long)m * g.ldcf + n) = s;
                }
            }
        }
        if (!transposed) return;
        __syncthreads();
        constexpr int CPT = T / 8;
#pragma unroll
        for (int q = 0; q < T * CPT / kThreads; ++q) {
            const int c = t + kThreads * q, row = c / CPT, col = (c % CPT) * 8;
            if (n0 + row < g.n_real && m0 + col < g.M)
                *reinterpret_cast<u32x4*>(g.Ct + (long)(n0 + row) * g.ldct + m0 + col) =
                    *reinterpret_cast<const u32x4*>(&Bs[row * LDT + col]);
        }
        return;
    }
    double lsum = 0.0;   // linear output with the loss: this thread's squares of Y - T
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int mb = m0 + wm + i * 16 + (lane >> 4) * 4;   // rows mb .. mb + 3
            const int n = n0 + wn + j * 16 + (lane & 15);
            if (n >= g.N) continue;
            if (EPI == kPartial) {
                if (n >= g.n_real) continue;
                float* out = g.Cf + bz * g.part_stride;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (mb + r < g.M) out[(long)(mb + r) * g.ldcf + n] = acc[i][j][r];
            } else if (!g.T) {
                if (n >= g.n_real) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (mb + r < g.M) g.Cf[(long)(mb + r) * g.ldcf + n] = acc[i][j][r] + g.bias[n];
            } else {
                // M is a multiple of 64 here (padded minibatch rows)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = mb + r;
                    float d = 0.0f;
                    if (n < g.n_real) {
                        const float y = acc[i][j][r] + g.bias[n];
                        g.Cf[(long)row * g.ldcf + n] = y;
                        if (row < g.rows) {
                            d = y - side[i][j][r];
                            lsum += (double)d * (double)d;
                        }
                    }
                    // rows * n_real formed in float (one rounding of the exact product, as the
                    // integer product's conversion would give) cannot overflow 32 bits
                    const bf16 v = (bf16)(2.0f * d / ((float)g.rows * (float)g.n_real));
                    g.dY[(long)row * g.lddy + n] = v;
                    if (n < g.n_real) g.dYt[(long)n * g.lddyt + row] = v;
                }
            }
        }
    if (EPI == kLinear && g.T) {
        // the tile's loss partial, summed over the workgroup in a fixed order (the K-loop
        // ended with a barrier, so As is free)
        double* red = reinterpret_cast<double*>(As);
        red[t] = lsum;
        __syncthreads();
        for (int w = kThreads / 2; w > 0; w >>= 1) {
            if (t < w) red[t] += red[t + w];
            __syncthreads();
        }
        if (t == 0) g.loss_part[by * g.nbx + bx] = red[0];
    }
}

template <int EPI, int BK, int T>
__global__ void __launch_bounds__(kThreads) gemm_kernel(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) bf16 As[kLdsElems<BK, T>];
    __shared__ __attribute__((aligned(16))) bf16 Bs[kLdsElems<BK, T>];
    gemm_tile<EPI, BK, T>(g, blockIdx.x, blockIdx.y, blockIdx.z, As, Bs);
}

// The output layer, of at most 16 columns: a wavefront per 16 rows, which loads its operands straight
// into the MFMA's registers, kThinStages groups of 8 K-steps ahead.  A 64 x 64 tile would be 1/21
// used and leave a workgroup alone with its loads on 16 of 256 CUs (1024 rows: 11.2 -> 5.2 us).
// The epilogue is gemm_tile's linear one, a loss partial per 16 rows.
constexpr int kThinStages = 3;

__global__ void __launch_bounds__(64) thin_linear_kernel(GemmArgs g) {
    const int lane = threadIdx.x, r16 = lane & 15, k8 = (lane >> 4) * 8;
    const int m0 = blockIdx.x * 16, mb = m0 + (lane >> 4) * 4, n = r16;
    const bf16* pa = g.A + (long)(m0 + r16) * g.lda + k8;   // M is a multiple of 64, N of 32
    const bf16* pb = g.B + (long)r16 * g.ldb + k8;
    const int nk = g.K / 32, groups = (nk + 7) / 8;
    bf16x8 a[kThinStages][8], b[kThinStages][8];
    auto load = [&](int slot, int group) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = min(group * 8 + u, nk - 1) * 32;   // past the last step: that one again, unused
            a[slot][u] = *reinterpret_cast<const bf16x8*>(pa + k);
            b[slot][u] = *reinterpret_cast<const bf16x8*>(pb + k);
        }
    };
    const float bias = n < g.n_real ? g.bias[n] : 0.0f;
    float tgt[4] = {};
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (g.T && n < g.n_real && mb + r < g.rows) tgt[r] = g.T[(long)(mb + r) * g.n_real + n];
#pragma unroll
    for (int d = 0; d < kThinStages; ++d)
        if (d < groups) load(d, d);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int g0 = 0; g0 < groups; g0 += kThinStages)
#pragma unroll
        for (int d = 0; d < kThinStages; ++d) {
            if (g0 + d >= groups) break;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if ((g0 + d) * 8 + u < nk) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[d][u], b[d][u], acc, 0, 0, 0);
            if (g0 + d + kThinStages < groups) load(d, g0 + d + kThinStages);
        }
    if (!g.T) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (n < g.n_real) g.Cf[(long)(mb + r) * g.ldcf + n] = acc[r] + bias;
        return;
    }
    double lsum = 0.0;
    bf16 v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = mb + r;
        float d = 0.0f;
        if (n < g.n_real) {
            const float y = acc[r] + bias;
            g.Cf[(long)row * g.ldcf + n] = y;
            if (row < g.rows) {
                d = y - tgt[r];
                lsum += (double)d * (double)d;
            }
        }
        v[r] = (bf16)(2.0f * d / ((float)g.rows * (float)g.n_real));
        for (int c = n; c < g.N; c += 16) g.dY[(long)row * g.lddy + c] = c == n ? v[r] : (bf16)0.0f;
    }
    if (n < g.n_real)
        *reinterpret_cast<uint2*>(g.dYt + (long)n * g.lddyt + mb) = uint2{pack2(v[0], v[1]), pack2(v[2], v[3])};
    for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, 64);
    if (lane == 0) g.loss_part[blockIdx.x] = lsum;
}

// Two independent products in one launch (the backward's weight gradient of a layer and the
// gradient into its input both read only that layer's dZ): workgroups below g1's tile count
// take g1's tiles, the rest g2's, so both run side by side on the chip without a second
// stream.  Tiles are numbered column fastest, then row, then split.
template <int E1, int BK1, int E2, int BK2>
__global__ void __launch_bounds__(kThreads) gemm_pair_kernel(GemmArgs g1, GemmArgs g2) {
    constexpr int BK = BK1 > BK2 ? BK1 : BK2;
    __shared__ __attribute__((aligned(16))) bf16 As[kLdsElems<BK, kTile>];
    __shared__ __attribute__((aligned(16))) bf16 Bs[kLdsElems<BK, kTile>];
    int tile = blockIdx.x;
    if (tile < g1.tiles) {
        gemm_tile<E1, BK1, kTile>(g1, tile % g1.nbx, (tile / g1.nbx) % g1.nby, tile / (g1.nbx * g1.nby), As, Bs);
    } else {
        tile -= g1.tiles;
        gemm_tile<E2, BK2, kTile>(g2, tile % g2.nbx, (tile / g2.nbx) % g2.nby, tile / (g2.nbx * g2.nby), As, Bs);
    }
}

// Sum of `splits` FP32 partials in split order: out[i] = part[0][i] + part[1][i] + ...
__global__ void splitk_sum_kernel(const float* part, long stride, int splits, float* out, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float s = part[i];
    for (int z = 1; z < splits; ++z) s += part[z * stride + i];
    out[i] = s;
}

// Where each layer's weights sit in the parameter vector and in the two BF16 shadows.
struct ShadowMap {
    long off_w[4], off_b[4];
    int K[4], N[4], Kp[4], Np[4];
    bf16* w[4];    // [Kp][Np]: W as stored (input-gradient products)
    bf16* wt[4];   // [Np][Kp]: W^T (forward products)
};

__device__ __forceinline__ void write_shadow(const ShadowMap& s, long i, float v) {
#pragma unroll
    for (int l = 0; l < 4; ++l)
        if (i >= s.off_w[l] && i < s.off_b[l]) {
            const long q = i - s.off_w[l];
            const int k = (int)(q / s.N[l]), n = (int)(q % s.N[l]);
            s.w[l][(long)k * s.Np[l] + n] = (bf16)v;
            s.wt[l][(long)n * s.Kp[l] + k] = (bf16)v;
        }
}

// Adam on the FP32 master copy; refreshes the BF16 shadows of the weight entries.  The
// gradient is the sum of `splits` partial gradients laid out like the parameters, `stride`
// apart, added in split order (the order splitk_sum_kernel uses).  A workgroup takes 32 rows by 64
// columns of one layer's weights, so that both shadows are written along their rows (the transposed one through
// LDS), or, after the tiles, one layer's biases.  Memory-bound: 36 B a parameter with two
// splits; 1.26 M parameters 15.9 -> 13.3 us (one thread per parameter, a 64-bit division for its row
// and column and a transposed shadow scattered 2 bytes at a time).
struct AdamMap {
    ShadowMap s;
    int first[5];   // first workgroup of each layer's tiles; first[4]: of the biases
};

__global__ void __launch_bounds__(256)
adam_kernel(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v, const float* __restrict__ grad,
            int splits, long stride, AdamMap a, float lr, float b1, float b2, float eps, float c1, float c2) {
    constexpr int TK = 32, PER = TK * 64 / 256;
    __shared__ __attribute__((aligned(16))) bf16 tile[64][TK + 8];   // [n][k]
    const int t = threadIdx.x;
    int blk = blockIdx.x;
    auto update = [&](long i, float gi, float mi, float vi, float pi) {
        mi = b1 * mi + (1.0f - b1) * gi;
        vi = b2 * vi + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        pi = pi - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        p[i] = pi;
        return pi;
    };
    if (blk >= a.first[4]) {
        const int l = blk - a.first[4];
        for (int n = t; n < a.s.N[l]; n += 256) {
            const long i = a.s.off_b[l] + n;
            float gi = grad[i];
            for (int z = 1; z < splits; ++z) gi += grad[z * stride + i];
            update(i, gi, m[i], v[i], p[i]);
        }
        return;
    }
    int l = 0;
    while (l < 3 && blk >= a.first[l + 1]) ++l;
    blk -= a.first[l];
    const int K = a.s.K[l], N = a.s.N[l], Kp = a.s.Kp[l], Np = a.s.Np[l];
    const int tn = (N + 63) / 64, k0 = blk / tn * TK, n0 = blk % tn * 64;
    const int nl = t & 63, n = n0 + nl;
    // every load first: a thread's elements would otherwise wait for memory one after the other
    float gi[PER], mi[PER], vi[PER], pi[PER];
    const long i0 = a.s.off_w[l] + (long)(k0 + (t >> 6)) * N + n, di = 4l * N;
    const int have = n < N ? (min(K - k0, TK) - (t >> 6) + 3) / 4 : 0;   // this thread's rows: t / 64, + 4, ...
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (u < have) {
            const long i = i0 + u * di;
            gi[u] = grad[i];
            mi[u] = m[i];
            vi[u] = v[i];
            pi[u] = p[i];
        }
    for (int z = 1; z < splits; ++z)
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (u < have) gi[u] += grad[z * stride + i0 + u * di];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int kl = (t >> 6) + 4 * u;
        bf16 w = (bf16)0.0f;
        if (u < have) {
            w = (bf16)update(i0 + u * di, gi[u], mi[u], vi[u], pi[u]);
            a.s.w[l][(long)(k0 + kl) * Np + n] = w;
        }
        tile[nl][kl] = w;
    }
    __syncthreads();
    // 16-byte pieces of the transposed tile's rows
    const int r = t >> 2, c = (t & 3) * 8;
    bf16* const to = a.s.wt[l] + (long)(n0 + r) * Kp + k0 + c;
    if (n0 + r >= N) return;
    if (k0 + c + 8 <= K) *reinterpret_cast<u32x4*>(to) = *reinterpret_cast<const u32x4*>(&tile[r][c]);
    else
        for (int u = 0; u < 8 && k0 + c + u < K; ++u) to[u] = tile[r][c + u];
}

__global__ void shadow_kernel(const float* p, ShadowMap sm, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) write_shadow(sm, i, p[i]);
}

// Minibatch rows r < padded_rows: X_b[r][c] = bf16(X[src][c]) (zero beyond n_in and beyond
// `rows`), X_t[c][r] for c < n_in (X_t null: left out), T_b[r] = T[src]; src = idx[r], or r when idx is
// NULL.  A workgroup takes 16 rows (padded_rows is a multiple of 64) and 64 columns and turns them
// in LDS.
__global__ void __launch_bounds__(256)
gather_kernel(const float* __restrict__ X, const float* __restrict__ T, const int* __restrict__ idx,
              bf16* __restrict__ Xb, int ldx, bf16* __restrict__ Xt, long ldt, float* __restrict__ Tb, int rows,
              int n_in, int n_out) {
    __shared__ __attribute__((aligned(16))) bf16 turned[64][24];
    const int t = threadIdx.x, r0 = blockIdx.x * 16, rl = t >> 4, r = r0 + rl;
    auto from = [&](int row) { return row < rows ? (idx ? (long)idx[row] : (long)row) : -1; };
    const long src = from(r);
    const int cl = (t & 15) * 4, c0 = blockIdx.y * 64, c = c0 + cl;
    bf16 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = (src >= 0 && c + u < n_in) ? (bf16)X[src * n_in + c + u] : (bf16)0.0f;
    if (c < ldx) *reinterpret_cast<uint2*>(Xb + (long)r * ldx + c) = uint2{pack2(v[0], v[1]), pack2(v[2], v[3])};
    if (T && blockIdx.y == 0)
        for (int q = t; q < 16 * n_out; q += 256) {
            const long s = from(r0 + q / n_out);
            Tb[(long)r0 * n_out + q] = s >= 0 ? T[s * n_out + q % n_out] : 0.0f;
        }
    if (!Xt) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) turned[cl + u][rl] = v[u];
    __syncthreads();
    const int cc = t >> 1, h = (t & 1) * 8;
    if (t < 128 && c0 + cc < n_in)
        *reinterpret_cast<u32x4*>(Xt + (long)(c0 + cc) * ldt + r0 + h) = *reinterpret_cast<const u32x4*>(&turned[cc][h]);
}

__global__ void fill_kernel(bf16* p, long n, float v) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (bf16)v;
}

uint64_t splitmix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

int pad_width(int w) { return (w + kWidthPad - 1) / kWidthPad * kWidthPad; }

}  // namespace

using cronos::fail;

#define HIP_TRY(expr)                                                                             \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) return fail(CRONOS_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

struct cronos_mlp_t {
    int sizes[5];
    int wp[5];             // widths padded to multiples of 32
    int max_rows = 0;      // padded to a multiple of 64; row pitch of every transposed buffer
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    long n_params = 0;
    long off_w[4], off_b[4];
    float *p = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;
    bf16 *w[4] = {}, *wt[4] = {};      // BF16 shadows [wp[l]][wp[l+1]] and [wp[l+1]][wp[l]]
    ShadowMap smap;
    int step = 0;
    // activations for max_rows rows (row-major [rows][width]; transposed [width (+1)][max_rows])
    float* xin = nullptr;              // [rows][sizes[0]] FP32 staging of uploaded inputs
    bf16* x = nullptr;                 // [rows][wp[0]]
    bf16* xt = nullptr;                // [sizes[0] + 1][max_rows], last row ones
    float* slope[3] = {};              // [rows][wp[l+1]] gelu'(Z_l), kept by the forward for the backward
    bf16* h[3] = {};
    bf16* ht[3] = {};                  // [sizes[l+1] + 1][max_rows], last row ones
    float* y = nullptr;                // [rows][sizes[4]]
    float* t = nullptr;
    bf16* dy = nullptr;                // [rows][wp[4]]
    bf16* dyt = nullptr;               // [sizes[4]][max_rows]
    bf16* dz[3] = {};                  // [rows][wp[l+1]]
    bf16* dzt[3] = {};                 // [sizes[l+1]][max_rows]
    float* part_w = nullptr;           // [splits][n_params] split-K partials of the weight gradients
    int grad_splits = 1;               // partials Adam adds (1: the gradient is in grad)
    double* part = nullptr;            // loss partials of one minibatch: [loss_parts(max_rows)]
    // training data
    float* data_x = nullptr;
    float* data_t = nullptr;
    int* idx = nullptr;
    long data_rows = 0;
    double* epoch_part = nullptr;      // loss partials of the last epoch's minibatches, one after the other
    size_t epoch_part_cap = 0;
};

namespace {

// Tile counts of g over `splits` K-chunks, and the K-step it takes (64 or 32: the deeper that
// divides K and the chunk).
int prepare(GemmArgs& g, int splits, int tile = kTile) {
    g.nbx = (g.N + tile - 1) / tile;
    g.nby = (g.M + tile - 1) / tile;
    g.tiles = g.nbx * g.nby * splits;
    if (splits == 1) g.k_chunk = g.K;
    return g.K % 64 == 0 && g.k_chunk % 64 == 0 ? 64 : 32;
}

template <int EPI>
hipError_t gemm(hipStream_t st, GemmArgs g, int splits = 1) {
    const int bk = prepare(g, splits);
    const dim3 grid(g.nbx, g.nby, splits);
    if (bk == 64)
        hipLaunchKernelGGL((gemm_kernel<EPI, 64, kTile>), grid, dim3(kThreads), 0, st, g);
    else
        hipLaunchKernelGGL((gemm_kernel<EPI, 32, kTile>), grid, dim3(kThreads), 0, st, g);
    return hipGetLastError();
}

// A hidden layer's forward product.  A 128 x 128 tile does four times the arithmetic for twice the
// operand bytes of a 64 x 64 one, but leaves a CU one workgroup where two small ones share it: it pays
// from about two rounds of small tiles on.  Measured, small / wide (us): 2048 x 768 (384 small tiles)
// 10.3 / 12.9, 4096 x 768 (768) 14.0 / 14.1, 8192 x 512 (1024) 15.5 / 12.6.
constexpr int kWideTiles = 1000;

hipError_t launch_forward(hipStream_t st, GemmArgs g) {
    if (prepare(g, 1) < 64 || g.tiles < kWideTiles) return gemm<kFwdGelu>(st, g);
    prepare(g, 1, 128);
    hipLaunchKernelGGL((gemm_kernel<kFwdGelu, 64, 128>), dim3(g.nbx, g.nby), dim3(kThreads), 0, st, g);
    return hipGetLastError();
}

// Output layers of at most this many columns take thin_linear_kernel.
constexpr int kThinColumns = 16;

// Loss partials that the output layer's product leaves for `rows` rows of n_out columns: one per
// wavefront of the narrow kernel, else one per tile.  Not falling in either argument.
size_t loss_parts(int n_out, int rows) {
    const int padded = (rows + 63) / 64 * 64;
    if (n_out <= kThinColumns) return (size_t)padded / 16;
    return (size_t)(padded / kTile) * (size_t)((pad_width(n_out) + kTile - 1) / kTile);
}

// The output layer's product; with the loss, into g.loss_part, which has room for `room` partials.
cronos_status launch_output(hipStream_t st, GemmArgs g, size_t room) {
    const bool thin = g.n_real <= kThinColumns;
    prepare(g, 1);
    const size_t parts = thin ? (size_t)g.M / 16 : (size_t)g.nbx * (size_t)g.nby;
    if (g.T && parts > room) return fail(CRONOS_EINVAL, "mlp: %zu loss partials, room for %zu", parts, room);
    if (thin) {
        hipLaunchKernelGGL(thin_linear_kernel, dim3(g.M / 16), dim3(64), 0, st, g);
        HIP_TRY(hipGetLastError());
    } else {
        HIP_TRY(gemm<kLinear>(st, g));
    }
    return CRONOS_OK;
}

template <int E1, int BK1, int E2>
void launch_pair2(hipStream_t st, const GemmArgs& g1, const GemmArgs& g2, int bk2) {
    const dim3 grid((unsigned)(g1.tiles + g2.tiles));
    if (bk2 == 64)
        hipLaunchKernelGGL((gemm_pair_kernel<E1, BK1, E2, 64>), grid, dim3(kThreads), 0, st, g1, g2);
    else
        hipLaunchKernelGGL((gemm_pair_kernel<E1, BK1, E2, 32>), grid, dim3(kThreads), 0, st, g1, g2);
}

// g1 over splits1 K-chunks and g2 (one chunk) in one launch.
template <int E1, int E2>
hipError_t gemm_pair(hipStream_t st, GemmArgs g1, int splits1, GemmArgs g2) {
    const int bk1 = prepare(g1, splits1), bk2 = prepare(g2, 1);
    if (bk1 == 64)
        launch_pair2<E1, 64, E2>(st, g1, g2, bk2);
    else
        launch_pair2<E1, 32, E2>(st, g1, g2, bk2);
    return hipGetLastError();
}

void free_mlp(cronos_mlp_t* q) {
    std::vector<void*> ptrs = {q->p, q->m, q->v, q->grad, q->xin, q->x, q->xt, q->y, q->t, q->dy, q->dyt, q->part_w,
                               q->part, q->data_x, q->data_t, q->idx, q->epoch_part};
    for (int l = 0; l < 4; ++l) {
        ptrs.push_back(q->w[l]);
        ptrs.push_back(q->wt[l]);
    }
    for (int l = 0; l < 3; ++l) {
        ptrs.push_back(q->slope[l]);
        ptrs.push_back(q->h[l]);
        ptrs.push_back(q->ht[l]);
        ptrs.push_back(q->dz[l]);
        ptrs.push_back(q->dzt[l]);
    }
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    if (q->own_stream && q->stream) (void)hipStreamDestroy(q->stream);
}

// Forward over `rows` (<= max_rows, padded to 64) rows already in q->x; with_loss: the output
// product's epilogue also forms the loss partials and dY from the targets in q->t, and the hidden
// layers keep what the backward products read (the activation's slopes, transposed activations).
// loss_part: where the loss partials go (loss_parts of them), with room for loss_room.
cronos_status forward_dev(cronos_mlp_t* q, int rows, bool with_loss, double* loss_part, size_t loss_room) {
    const int P = (rows + 63) / 64 * 64;
    const long R = q->max_rows;
    const bf16* in = q->x;
    for (int l = 0; l < 3; ++l) {
        GemmArgs g{};
        g.A = in;
        g.lda = q->wp[l];
        g.B = q->wt[l];
        g.ldb = q->wp[l];
        g.M = P;
        g.N = q->wp[l + 1];
        g.K = q->wp[l];
        g.n_real = q->sizes[l + 1];
        g.bias = q->p + q->off_b[l];
        g.Cf = with_loss ? q->slope[l] : nullptr;
        g.ldcf = q->wp[l + 1];
        g.Cb = q->h[l];
        g.ldcb = q->wp[l + 1];
        g.Ct = q->ht[l];
        g.ldct = R;
        HIP_TRY(launch_forward(q->stream, g));
        in = q->h[l];
    }
    GemmArgs g{};
    g.A = in;
    g.lda = q->wp[3];
    g.B = q->wt[3];
    g.ldb = q->wp[3];
    g.M = P;
    g.N = q->wp[4];
    g.K = q->wp[3];
    g.n_real = q->sizes[4];
    g.bias = q->p + q->off_b[3];
    g.Cf = q->y;
    g.ldcf = q->sizes[4];
    if (with_loss) {
        g.T = q->t;
        g.dY = q->dy;
        g.lddy = q->wp[4];
        g.dYt = q->dyt;
        g.lddyt = R;
        g.loss_part = loss_part;
        g.rows = rows;
    }
    return launch_output(q->stream, g, loss_room);
}

// Loss and gradients for `rows` rows whose inputs are in q->x / q->xt and targets in q->t.
// With more than one K-split the weight gradients stay as per-split partials (q->part_w,
// laid out like the parameters) for Adam to add, unless sum_grads asks for them in q->grad.
cronos_status backward_dev(cronos_mlp_t* q, int rows, bool sum_grads) {
    const int P = (rows + 63) / 64 * 64;
    const long R = q->max_rows;
    const int splits = (P + kSplitRows - 1) / kSplitRows;
    const bf16* dnext = q->dy;     // [P][wp[l+1]]
    const bf16* dnext_t = q->dyt;  // [sizes[l+1]][R]
    for (int l = 3; l >= 0; --l) {
        const int K = q->sizes[l], N = q->sizes[l + 1];
        // [dW_l; db_l] = [H_in^T; 1] dZ_l : (K + 1) x N, summed over the P rows
        GemmArgs g{};
        g.A = l ? q->ht[l - 1] : q->xt;
        g.lda = R;
        g.B = dnext_t;
        g.ldb = R;
        g.M = K + 1;
        g.N = N;
        g.K = P;
        g.k_chunk = kSplitRows;
        g.n_real = N;
        g.ldcf = N;
        if (splits == 1) {
            g.Cf = q->grad + q->off_w[l];
        } else {
            g.Cf = q->part_w + q->off_w[l];
            g.part_stride = q->n_params;
        }
        if (l == 0) HIP_TRY(gemm<kPartial>(q->stream, g, splits));
        if (l) {
            // dZ_{l-1} = (dZ_l W_l^T) * gelu'(Z_{l-1}), the slopes as the forward left them : (P x wp[l+1]) (wp[l+1] x wp[l])
            GemmArgs d{};
            d.A = dnext;
            d.lda = q->wp[l + 1];
            d.B = q->w[l];
            d.ldb = q->wp[l + 1];
            d.M = P;
            d.N = q->wp[l];
            d.K = q->wp[l + 1];
            d.n_real = K;
            d.Cb = q->dz[l - 1];
            d.ldcb = q->wp[l];
            d.Ct = q->dzt[l - 1];
            d.ldct = R;
            d.S = q->slope[l - 1];
            d.lds = q->wp[l];
            // both read dZ_l only: one launch for the pair
            HIP_TRY((gemm_pair<kPartial, kBwdGelu>(q->stream, g, splits, d)));
            dnext = q->dz[l - 1];
            dnext_t = q->dzt[l - 1];
        }
    }
    q->grad_splits = splits;
    if (splits > 1 && sum_grads) {
        hipLaunchKernelGGL(splitk_sum_kernel, dim3((unsigned)((q->n_params + 255) / 256)), dim3(256), 0, q->stream,
                           q->part_w, q->n_params, splits, q->grad, q->n_params);
        HIP_TRY(hipGetLastError());
        q->grad_splits = 1;
    }
    return CRONOS_OK;
}

// Rows of the minibatch from device arrays (idx == nullptr: the first `rows` rows in order).
// backward: the transposed rows as well, which only the backward reads.
cronos_status gather_rows(cronos_mlp_t* q, const float* X, const float* T, const int* idx, int rows, bool backward) {
    const int P = (rows + 63) / 64 * 64;
    hipLaunchKernelGGL(gather_kernel, dim3(P / 16, (q->wp[0] + 63) / 64), dim3(256), 0, q->stream, X, T, idx, q->x, q->wp[0],
                       backward ? q->xt : nullptr, (long)q->max_rows, q->t, rows, q->sizes[0], q->sizes[4]);
    HIP_TRY(hipGetLastError());
    return CRONOS_OK;
}

cronos_status upload_rows(cronos_mlp_t* q, const float* x, const float* t, int rows) {
    const int n_in = q->sizes[0], n_out = q->sizes[4];
    HIP_TRY(hipMemcpyAsync(q->xin, x, (size_t)rows * n_in * sizeof(float), hipMemcpyHostToDevice, q->stream));
    // targets: the loss reads rows below `rows` only
    if (t) HIP_TRY(hipMemcpyAsync(q->t, t, (size_t)rows * n_out * sizeof(float), hipMemcpyHostToDevice, q->stream));
    return gather_rows(q, q->xin, nullptr, nullptr, rows, t != nullptr);
}

cronos_status adam_dev(cronos_mlp_t* q, double lr, double b1, double b2, double eps) {
    q->step += 1;
    const float c1 = (float)(1.0 - std::pow(b1, q->step)), c2 = (float)(1.0 - std::pow(b2, q->step));
    const bool parts = q->grad_splits > 1;
    AdamMap a{q->smap, {}};
    for (int l = 0; l < 4; ++l) a.first[l + 1] = a.first[l] + (q->sizes[l] + 31) / 32 * ((q->sizes[l + 1] + 63) / 64);
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)(a.first[4] + 4)), dim3(256), 0, q->stream, q->p, q->m, q->v,
                       parts ? q->part_w : q->grad, parts ? q->grad_splits : 1, q->n_params, a, (float)lr, (float)b1,
                       (float)b2, (float)eps, c1, c2);
    HIP_TRY(hipGetLastError());
    return CRONOS_OK;
}

// The loss of `rows` rows from its partials (host copies).
double loss_of(const cronos_mlp_t* q, const double* parts, size_t count, int rows) {
    double s = 0.0;
    for (size_t k = 0; k < count; ++k) s += parts[k];
    return s / ((double)rows * q->sizes[4]);
}

double loss_from_parts(cronos_mlp_t* q, int rows, cronos_status* st) {
    const size_t nb = loss_parts(q->sizes[4], rows);
    std::vector<double> h(nb);
    *st = CRONOS_OK;
    if (hipMemcpyAsync(h.data(), q->part, nb * sizeof(double), hipMemcpyDeviceToHost, q->stream) != hipSuccess ||
        hipStreamSynchronize(q->stream) != hipSuccess) {
        *st = fail(CRONOS_EDEVICE, "mlp: loss read-back failed");
        return 0.0;
    }
    return loss_of(q, h.data(), nb, rows);
}

}  // namespace

extern "C" cronos_status cronos_mlp_create(const int32_t* sizes, const double* params, int32_t max_rows, int32_t device,
                                           void* stream, cronos_mlp* out) {
    cronos::clear_error();
    if (!sizes || !params || !out || max_rows < 1) return fail(CRONOS_EINVAL, "mlp_create: bad arguments");
    *out = nullptr;
    for (int l = 0; l < 5; ++l)
        if (sizes[l] < 1 || sizes[l] > 4096) return fail(CRONOS_EINVAL, "mlp_create: layer width out of range");
    if (max_rows > (1 << 20)) return fail(CRONOS_EINVAL, "mlp_create: max_rows above 2^20");
    auto* q = new (std::nothrow) cronos_mlp_t;
    if (!q) return fail(CRONOS_ENOMEM, "mlp_create: out of memory");
    for (int l = 0; l < 5; ++l) {
        q->sizes[l] = sizes[l];
        q->wp[l] = pad_width(sizes[l]);
    }
    q->max_rows = (max_rows + 63) / 64 * 64;
    q->device = device;
    long off = 0;
    for (int l = 0; l < 4; ++l) {
        q->off_w[l] = off;
        off += (long)sizes[l] * sizes[l + 1];
        q->off_b[l] = off;
        off += sizes[l + 1];
    }
    q->n_params = off;
    auto st = [&]() -> cronos_status {
        HIP_TRY(hipSetDevice(device));
        if (stream) {
            q->stream = (hipStream_t)stream;
        } else {
            HIP_TRY(hipStreamCreateWithFlags(&q->stream, hipStreamNonBlocking));
            q->own_stream = true;
        }
        const long n = q->n_params, R = q->max_rows;
        auto dmalloc = [&](auto** ptr, size_t count) -> hipError_t {
            return hipMalloc((void**)ptr, std::max<size_t>(count, 1) * sizeof(**ptr));
        };
        HIP_TRY(dmalloc(&q->p, n));
        HIP_TRY(dmalloc(&q->m, n));
        HIP_TRY(dmalloc(&q->v, n));
        HIP_TRY(dmalloc(&q->grad, n));
        for (int l = 0; l < 4; ++l) {
            const size_t cnt = (size_t)q->wp[l] * q->wp[l + 1];
            HIP_TRY(dmalloc(&q->w[l], cnt));
            HIP_TRY(dmalloc(&q->wt[l], cnt));
            HIP_TRY(hipMemsetAsync(q->w[l], 0, cnt * sizeof(bf16), q->stream));
            HIP_TRY(hipMemsetAsync(q->wt[l], 0, cnt * sizeof(bf16), q->stream));
            q->smap.off_w[l] = q->off_w[l];
            q->smap.off_b[l] = q->off_b[l];
            q->smap.K[l] = sizes[l];
            q->smap.N[l] = sizes[l + 1];
            q->smap.Kp[l] = q->wp[l];
            q->smap.Np[l] = q->wp[l + 1];
            q->smap.w[l] = q->w[l];
            q->smap.wt[l] = q->wt[l];
        }
        HIP_TRY(dmalloc(&q->xin, R * sizes[0]));
        HIP_TRY(dmalloc(&q->x, R * q->wp[0]));
        HIP_TRY(dmalloc(&q->xt, (sizes[0] + 1) * R));
        for (int l = 0; l < 3; ++l) {
            HIP_TRY(dmalloc(&q->slope[l], R * q->wp[l + 1]));
            HIP_TRY(dmalloc(&q->h[l], R * q->wp[l + 1]));
            HIP_TRY(dmalloc(&q->ht[l], (sizes[l + 1] + 1) * R));
            HIP_TRY(dmalloc(&q->dz[l], R * q->wp[l + 1]));
            HIP_TRY(dmalloc(&q->dzt[l], sizes[l + 1] * R));
        }
        HIP_TRY(dmalloc(&q->y, R * sizes[4]));
        HIP_TRY(dmalloc(&q->t, R * sizes[4]));
        HIP_TRY(dmalloc(&q->dy, R * q->wp[4]));
        HIP_TRY(dmalloc(&q->dyt, sizes[4] * R));
        HIP_TRY(dmalloc(&q->part, loss_parts(sizes[4], q->max_rows)));
        // split-K partials of the weight gradients at max_rows rows, laid out like the parameters
        const int splits = (int)((R + kSplitRows - 1) / kSplitRows);
        if (splits > 1) HIP_TRY(dmalloc(&q->part_w, (size_t)splits * n));
        // the appended row of ones of every transposed layer input
        auto ones = [&](bf16* base, int row) -> hipError_t {
            hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, q->stream, base + (long)row * R, R,
                               1.0f);
            return hipGetLastError();
        };
        HIP_TRY(ones(q->xt, sizes[0]));
        for (int l = 0; l < 3; ++l) HIP_TRY(ones(q->ht[l], sizes[l + 1]));
        std::vector<float> hp(n), zero(n, 0.0f);
        for (long i = 0; i < n; ++i) hp[i] = (float)params[i];
        HIP_TRY(hipMemcpyAsync(q->p, hp.data(), n * sizeof(float), hipMemcpyHostToDevice, q->stream));
        HIP_TRY(hipMemcpyAsync(q->m, zero.data(), n * sizeof(float), hipMemcpyHostToDevice, q->stream));
        HIP_TRY(hipMemcpyAsync(q->v, zero.data(), n * sizeof(float), hipMemcpyHostToDevice, q->stream));
        HIP_TRY(hipMemcpyAsync(q->grad, zero.data(), n * sizeof(float), hipMemcpyHostToDevice, q->stream));
        hipLaunchKernelGGL(shadow_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, q->stream, q->p, q->smap, n);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipStreamSynchronize(q->stream));
        return CRONOS_OK;
    }();
    if (st != CRONOS_OK) {
        free_mlp(q);
        delete q;
        return st;
    }
    *out = q;
    return CRONOS_OK;
}

extern "C" void cronos_mlp_destroy(cronos_mlp q) {
    if (!q) return;
    (void)hipSetDevice(q->device);
    (void)hipStreamSynchronize(q->stream);
    free_mlp(q);
    delete q;
}

extern "C" cronos_status cronos_mlp_get_params(cronos_mlp q, double* params) {
    if (!q || !params) return fail(CRONOS_EINVAL, "mlp_get_params: NULL argument");
    std::vector<float> hp(q->n_params);
    HIP_TRY(hipSetDevice(q->device));
    HIP_TRY(hipMemcpyAsync(hp.data(), q->p, q->n_params * sizeof(float), hipMemcpyDeviceToHost, q->stream));
    HIP_TRY(hipStreamSynchronize(q->stream));
    for (long i = 0; i < q->n_params; ++i) params[i] = hp[i];
    return CRONOS_OK;
}

extern "C" cronos_status cronos_mlp_forward(cronos_mlp q, const float* x, int64_t rows, float* y) {
    cronos::clear_error();
    if (!q || !x || !y || rows < 0) return fail(CRONOS_EINVAL, "mlp_forward: bad arguments");
    HIP_TRY(hipSetDevice(q->device));
    const int n_out = q->sizes[4];
    for (int64_t r0 = 0; r0 < rows; r0 += q->max_rows) {
        const int r = (int)std::min<int64_t>(q->max_rows, rows - r0);
        cronos_status st = upload_rows(q, x + r0 * q->sizes[0], nullptr, r);
        if (st != CRONOS_OK) return st;
        st = forward_dev(q, r, false, nullptr, 0);
        if (st != CRONOS_OK) return st;
        HIP_TRY(hipMemcpyAsync(y + r0 * n_out, q->y, (size_t)r * n_out * sizeof(float), hipMemcpyDeviceToHost, q->stream));
        HIP_TRY(hipStreamSynchronize(q->stream));
    }
    return CRONOS_OK;
}

extern "C" cronos_status cronos_mlp_loss_grad(cronos_mlp q, const float* x, const float* t, int32_t rows, double* loss,
                                              double* grads) {
    cronos::clear_error();
    if (!q || !x || !t || rows < 1 || rows > q->max_rows) return fail(CRONOS_EINVAL, "mlp_loss_grad: bad arguments");
    HIP_TRY(hipSetDevice(q->device));
    cronos_status st = upload_rows(q, x, t, rows);
    if (st == CRONOS_OK) st = forward_dev(q, rows, true, q->part, loss_parts(q->sizes[4], q->max_rows));
    if (st == CRONOS_OK) st = backward_dev(q, rows, true);
    if (st != CRONOS_OK) return st;
    const double l = loss_from_parts(q, rows, &st);
    if (st != CRONOS_OK) return st;
    if (loss) *loss = l;
    if (grads) {
        std::vector<float> hg(q->n_params);
        HIP_TRY(hipMemcpyAsync(hg.data(), q->grad, q->n_params * sizeof(float), hipMemcpyDeviceToHost, q->stream));
        HIP_TRY(hipStreamSynchronize(q->stream));
        for (long i = 0; i < q->n_params; ++i) grads[i] = hg[i];
    }
    return CRONOS_OK;
}

extern "C" cronos_status cronos_mlp_adam(cronos_mlp q, double lr, double beta1, double beta2, double eps) {
    cronos::clear_error();
    if (!q) return fail(CRONOS_EINVAL, "mlp_adam: NULL handle");
    HIP_TRY(hipSetDevice(q->device));
    cronos_status st = adam_dev(q, lr, beta1, beta2, eps);
    if (st != CRONOS_OK) return st;
    HIP_TRY(hipStreamSynchronize(q->stream));
    return CRONOS_OK;
}

extern "C" cronos_status cronos_mlp_train(cronos_mlp q, const float* x, const float* t, int64_t rows, int32_t batch,
                                          int32_t epochs, double lr, double lr_final, uint64_t seed, double* epoch_loss) {
    cronos::clear_error();
    if (!q || !x || !t || rows < 1 || batch < 1 || batch > q->max_rows || epochs < 0 || !(lr >= 0.0) ||
        !(lr_final >= 0.0))
        return fail(CRONOS_EINVAL, "mlp_train: bad arguments");
    HIP_TRY(hipSetDevice(q->device));
    const int n_in = q->sizes[0], n_out = q->sizes[4];
    if (q->data_rows != rows) {
        if (q->data_x) (void)hipFree(q->data_x);
        if (q->data_t) (void)hipFree(q->data_t);
        if (q->idx) (void)hipFree(q->idx);
        q->data_x = nullptr;
        q->data_t = nullptr;
        q->idx = nullptr;
        q->data_rows = 0;
        HIP_TRY(hipMalloc((void**)&q->data_x, (size_t)rows * n_in * sizeof(float)));
        HIP_TRY(hipMalloc((void**)&q->data_t, (size_t)rows * n_out * sizeof(float)));
        HIP_TRY(hipMalloc((void**)&q->idx, (size_t)rows * sizeof(int)));
        q->data_rows = rows;
    }
    HIP_TRY(hipMemcpyAsync(q->data_x, x, (size_t)rows * n_in * sizeof(float), hipMemcpyHostToDevice, q->stream));
    HIP_TRY(hipMemcpyAsync(q->data_t, t, (size_t)rows * n_out * sizeof(float), hipMemcpyHostToDevice, q->stream));
    // learning rate: cosine from lr to lr_final over all minibatch steps (constant if equal)
    const int64_t per_epoch = (rows + batch - 1) / batch, last = std::max<int64_t>(1, per_epoch * epochs - 1);
    // loss partials of the last epoch, read back once at its end
    const size_t parts_cap = (size_t)per_epoch * loss_parts(n_out, (int)std::min<int64_t>(batch, rows));
    if (q->epoch_part_cap < parts_cap) {
        if (q->epoch_part) (void)hipFree(q->epoch_part);
        q->epoch_part = nullptr;
        q->epoch_part_cap = 0;
        HIP_TRY(hipMalloc((void**)&q->epoch_part, parts_cap * sizeof(double)));
        q->epoch_part_cap = parts_cap;
    }
    // epoch order: Fisher-Yates driven by SplitMix64(seed, epoch, i); the next epoch's is drawn while the
    // device works on this one
    std::vector<int> perm[2];
    auto draw_order = [&](int e) {
        std::vector<int>& o = perm[e & 1];
        o.resize(rows);
        for (int64_t i = 0; i < rows; ++i) o[i] = (int)i;
        const uint64_t base = splitmix64(seed ^ (0x5851F42D4C957F2Dull * (uint64_t)(e + 1)));
        for (int64_t i = rows - 1; i > 0; --i) std::swap(o[i], o[(int64_t)(splitmix64(base ^ (uint64_t)i) % (uint64_t)(i + 1))]);
    };
    if (epochs > 0) draw_order(0);
    int64_t step = 0;
    for (int e = 0; e < epochs; ++e) {
        const bool final_epoch = e == epochs - 1;
        HIP_TRY(hipMemcpyAsync(q->idx, perm[e & 1].data(), rows * sizeof(int), hipMemcpyHostToDevice, q->stream));
        size_t parts = 0;   // loss partials of the last epoch's minibatches so far
        for (int64_t b0 = 0; b0 < rows; b0 += batch) {
            const int r = (int)std::min<int64_t>(batch, rows - b0);
            cronos_status st = gather_rows(q, q->data_x, q->data_t, q->idx + b0, r, true);
            if (st == CRONOS_OK) st = final_epoch ? forward_dev(q, r, true, q->epoch_part + parts, q->epoch_part_cap - parts)
                                               : forward_dev(q, r, true, q->part, loss_parts(n_out, q->max_rows));
            if (st == CRONOS_OK) st = backward_dev(q, r, false);
            const double lr_t = lr_final + 0.5 * (lr - lr_final) * (1.0 + std::cos(M_PI * (double)step++ / (double)last));
            if (st == CRONOS_OK) st = adam_dev(q, lr_t, 0.9, 0.999, 1e-8);
            if (st != CRONOS_OK) return st;
            if (final_epoch) parts += loss_parts(n_out, r);
        }
        if (!final_epoch) {
            draw_order(e + 1);
            HIP_TRY(hipStreamSynchronize(q->stream));   // this epoch's order is rewritten after the next
            continue;
        }
        std::vector<double> h(parts);
        HIP_TRY(hipMemcpyAsync(h.data(), q->epoch_part, parts * sizeof(double), hipMemcpyDeviceToHost, q->stream));
        HIP_TRY(hipStreamSynchronize(q->stream));
        double sum = 0.0;
        size_t at = 0;
        for (int64_t b = 0; b < per_epoch; ++b) {
            const int r = (int)std::min<int64_t>(batch, rows - b * batch);
            const size_t count = loss_parts(n_out, r);
            sum += loss_of(q, h.data() + at, count, r) * r;
            at += count;
        }
        if (epoch_loss) *epoch_loss = sum / (double)rows;
    }
    return CRONOS_OK;
}
