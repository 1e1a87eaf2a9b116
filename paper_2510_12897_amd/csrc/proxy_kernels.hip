// gfx950 kernels of the learned warm-start proxy: a multilayer perceptron
// that maps bus loads to (vm, va, pg, qg), trained with a penalty on the
// FP64 constraint violation that the callback kernels compute.
//
//  - prox_gemm / prox_gemm_mixed: C[M,N] = A[M,K] B[K,N] on the matrix
//    cores (v_mfma_f32_32x32x16_bf16), FP32 accumulation: each operand is
//    either FP32 in memory, rounded to BF16 (nearest even) when staged into
//    LDS, or already BF16 (the MLP's weight copy and hidden activations);
//    optional fused epilogue bias + exact GELU (FP32 or BF16 output), staged
//    through LDS for whole-row vector stores.  Two forms of the same products
//    in the same order: the tiled one (gemm_tile.h: direct-to-LDS copies,
//    several k tiles in flight) where the operands allow it, else the
//    register-staged one below (128x128 or 128x64 block tile, BK = 64, four
//    waves, one k tile in flight in registers).
//  - prox_gemm_gelu_bwd: the dh product with the GELU backward of the layer
//    below and the bias gradient's first column-sum pass in its epilogue.
//  - the fused loss (prox_loss_fused): the whole FP64 side of a sample in one
//    workgroup's LDS (squashing, arc flows, rows, penalty, Cvio, d loss / d z).
//  - elementwise / reduction kernels: GELU backward, deterministic column
//    sums (bias gradient), Adam (also with its step count on the device and
//    a BF16 copy of the parameters, 16-byte accesses where aligned), the
//    samples' loads and features, output squashing into the variable
//    bounds and its backward (also fused with the objective and loss-weight
//    step), the penalty loss with its constraint weights, and the chain
//    weights that carry the arc-flow gradient back to the voltages.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "dev_model.h"
#include "gemm_tile.h"
#include "proxy_kernels.h"

namespace opf {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int BM = 128, BK = 64;  // block tile rows (of A / C) and k depth; columns: 128 or 64
constexpr int GEMM_THREADS = 256;
constexpr int kXcd = 8;       // accelerator complex dies, each with its own L2
constexpr int kWideMin = 512; // 128-column tiles only when they give two workgroups per CU (256 CUs)

__device__ __forceinline__ __bf16 to_bf16(float f) { return (__bf16)f; }  // round to nearest even

__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float x) {
    // d/dx x Phi(x) = Phi(x) + x phi(x)
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// LDS operand tile: 128 rows (i of A, j of B) of BK = 64 BF16 values, eight
// 16-byte chunks of 8 k values per row.  Chunk c of row r sits at position
// c ^ ((r >> 1) & 7): the fragment reads (16 consecutive rows, one chunk) and
// the row-wise tile stores then fall on distinct banks.
__device__ __forceinline__ int lds_at(int r, int c) { return r * BK + ((c ^ ((r >> 1) & 7)) << 3); }

__device__ __forceinline__ bf16x8 pack8(float a0, float a1, float a2, float a3, float a4, float a5, float a6,
                                        float a7) {
    return (bf16x8){to_bf16(a0), to_bf16(a1), to_bf16(a2), to_bf16(a3),
                    to_bf16(a4), to_bf16(a5), to_bf16(a6), to_bf16(a7)};
}

// Global loads of one ROWS x BK operand tile (rows r0.., k0..; ROWS = 128 or
// 64), ROWS / 8 floats per thread, zero outside rows < nrows, k < kend.
// Sizes are multiples of 4, so each float4 is wholly inside or outside.
//  KCONT: element (r, k) at P[r * ld + k]; thread t holds row t / 8 + 32 q,
//         k = 8 (t % 8) .. + 8 as v[2q], v[2q + 1].
//  else:  element (r, k) at P[k * ld + r]; thread t holds the four rows
//         4 (t % G) .. + 4 (G = ROWS / 4 row groups) at the k values
//         K (t / G) + kk, K = 4 G / 8 (8 for 128 rows, 4 for 64), as v[kk]:
//         a coalesced row segment per k.
__device__ __forceinline__ float4 guarded_load(const float* __restrict__ base, const float* p, bool ok) {
    // an out-of-range load reads the (valid) first element and is discarded
    const float4 t = *reinterpret_cast<const float4*>(ok ? p : base);
    return ok ? t : make_float4(0.f, 0.f, 0.f, 0.f);
}

// Registers that stage one operand tile between its global load and its LDS
// store: FP32 operands as float4 (rounded to BF16 at the store); BF16
// operands as they are stored (k-contiguous: 8 k values of one row per
// 16-byte load; i-contiguous: 4 rows of one k per 8-byte load).
template <typename T, bool KCONT, int ROWS>
struct TileRegs {
    float4 v[ROWS / 16];
};
template <int ROWS>
struct TileRegs<__bf16, true, ROWS> {
    uint4 v[ROWS / 32];
};
template <int ROWS>
struct TileRegs<__bf16, false, ROWS> {
    uint2 v[ROWS / 16];
};

template <bool KCONT, int ROWS>
__device__ __forceinline__ void load_tile(const float* __restrict__ P, int ld, int nrows, int kend, int r0, int k0,
                                          TileRegs<float, KCONT, ROWS>& R) {
    float4 (&v)[ROWS / 16] = R.v;
    const int t = threadIdx.x;
    if (KCONT) {
        const int k = k0 + (t % 8) * 8;
#pragma unroll
        for (int q = 0; q < ROWS / 32; q++) {
            const int r = r0 + t / 8 + 32 * q;
            const float* p = P + (size_t)r * ld + k;
            v[2 * q] = guarded_load(P, p, r < nrows && k < kend);
            v[2 * q + 1] = guarded_load(P, p + 4, r < nrows && k + 4 < kend);
        }
    } else {
        constexpr int G = ROWS / 4, KPER = ROWS / 16;
        const int r = r0 + (t % G) * 4;
#pragma unroll
        for (int kk = 0; kk < KPER; kk++) {
            const int k = k0 + (t / G) * KPER + kk;
            v[kk] = guarded_load(P, P + (size_t)k * ld + r, r < nrows && k < kend);
        }
    }
}

// Rounds the loaded tile to BF16 and writes it to LDS as row chunks (the
// i-contiguous layout is transposed in registers: 16-byte chunks for 128
// rows, 8-byte half chunks for 64).
template <bool KCONT, int ROWS>
__device__ __forceinline__ void store_tile(__bf16* S, const TileRegs<float, KCONT, ROWS>& R) {
    const float4 (&v)[ROWS / 16] = R.v;
    const int t = threadIdx.x;
    if (KCONT) {
#pragma unroll
        for (int q = 0; q < ROWS / 32; q++) {
            const float4 a = v[2 * q], b = v[2 * q + 1];
            *reinterpret_cast<bf16x8*>(S + lds_at(t / 8 + 32 * q, t % 8)) =
                pack8(a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w);
        }
    } else if (ROWS == 128) {
        const int r = (t % 32) * 4, c = t / 32;
        *reinterpret_cast<bf16x8*>(S + lds_at(r + 0, c)) =
            pack8(v[0].x, v[1].x, v[2].x, v[3].x, v[4].x, v[5].x, v[6].x, v[7].x);
        *reinterpret_cast<bf16x8*>(S + lds_at(r + 1, c)) =
            pack8(v[0].y, v[1].y, v[2].y, v[3].y, v[4].y, v[5].y, v[6].y, v[7].y);
        *reinterpret_cast<bf16x8*>(S + lds_at(r + 2, c)) =
            pack8(v[0].z, v[1].z, v[2].z, v[3].z, v[4].z, v[5].z, v[6].z, v[7].z);
        *reinterpret_cast<bf16x8*>(S + lds_at(r + 3, c)) =
            pack8(v[0].w, v[1].w, v[2].w, v[3].w, v[4].w, v[5].w, v[6].w, v[7].w);
    } else {
        const int r = (t % 16) * 4, kq = t / 16;  // k = 4 kq .. + 4: half kq % 2 of chunk kq / 2
        const int c = kq / 2, h = (kq % 2) * 4;
        *reinterpret_cast<bf16x4*>(S + lds_at(r + 0, c) + h) =
            (bf16x4){to_bf16(v[0].x), to_bf16(v[1].x), to_bf16(v[2].x), to_bf16(v[3].x)};
        *reinterpret_cast<bf16x4*>(S + lds_at(r + 1, c) + h) =
            (bf16x4){to_bf16(v[0].y), to_bf16(v[1].y), to_bf16(v[2].y), to_bf16(v[3].y)};
        *reinterpret_cast<bf16x4*>(S + lds_at(r + 2, c) + h) =
            (bf16x4){to_bf16(v[0].z), to_bf16(v[1].z), to_bf16(v[2].z), to_bf16(v[3].z)};
        *reinterpret_cast<bf16x4*>(S + lds_at(r + 3, c) + h) =
            (bf16x4){to_bf16(v[0].w), to_bf16(v[1].w), to_bf16(v[2].w), to_bf16(v[3].w)};
    }
}

// BF16 operands: the same thread-to-element maps as the FP32 loads above.
// A k-contiguous operand has its k extent and leading dimension multiples
// of 8, so that every 16-byte load of 8 k values is wholly inside or outside.
template <bool KCONT, int ROWS>
__device__ __forceinline__ void load_tile(const __bf16* __restrict__ P, int ld, int nrows, int kend, int r0, int k0,
                                          TileRegs<__bf16, KCONT, ROWS>& R) {
    const int t = threadIdx.x;
    if constexpr (KCONT) {
        const int k = k0 + (t % 8) * 8;
#pragma unroll
        for (int q = 0; q < ROWS / 32; q++) {
            const int r = r0 + t / 8 + 32 * q;
            const bool ok = r < nrows && k < kend;
            const uint4 u = *reinterpret_cast<const uint4*>(ok ? P + (size_t)r * ld + k : P);
            R.v[q] = ok ? u : make_uint4(0u, 0u, 0u, 0u);
        }
    } else {
        constexpr int G = ROWS / 4, KPER = ROWS / 16;
        const int r = r0 + (t % G) * 4;
#pragma unroll
        for (int kk = 0; kk < KPER; kk++) {
            const int k = k0 + (t / G) * KPER + kk;
            const bool ok = r < nrows && k < kend;
            const uint2 u = *reinterpret_cast<const uint2*>(ok ? P + (size_t)k * ld + r : P);
            R.v[kk] = ok ? u : make_uint2(0u, 0u);
        }
    }
}

__device__ __forceinline__ uint32_t pack_lo(uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); }
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }

template <bool KCONT, int ROWS>
__device__ __forceinline__ void store_tile(__bf16* S, const TileRegs<__bf16, KCONT, ROWS>& R) {
    const int t = threadIdx.x;
    if constexpr (KCONT) {
#pragma unroll
        for (int q = 0; q < ROWS / 32; q++) *reinterpret_cast<uint4*>(S + lds_at(t / 8 + 32 * q, t % 8)) = R.v[q];
    } else if constexpr (ROWS == 128) {
        // thread: rows r .. r + 3 at k values 8 c .. 8 c + 7 (v[kk] = rows at k = 8 c + kk)
        const uint2* v = R.v;
        const int r = (t % 32) * 4, c = t / 32;
        *reinterpret_cast<uint4*>(S + lds_at(r + 0, c)) =
            make_uint4(pack_lo(v[0].x, v[1].x), pack_lo(v[2].x, v[3].x), pack_lo(v[4].x, v[5].x), pack_lo(v[6].x, v[7].x));
        *reinterpret_cast<uint4*>(S + lds_at(r + 1, c)) =
            make_uint4(pack_hi(v[0].x, v[1].x), pack_hi(v[2].x, v[3].x), pack_hi(v[4].x, v[5].x), pack_hi(v[6].x, v[7].x));
        *reinterpret_cast<uint4*>(S + lds_at(r + 2, c)) =
            make_uint4(pack_lo(v[0].y, v[1].y), pack_lo(v[2].y, v[3].y), pack_lo(v[4].y, v[5].y), pack_lo(v[6].y, v[7].y));
        *reinterpret_cast<uint4*>(S + lds_at(r + 3, c)) =
            make_uint4(pack_hi(v[0].y, v[1].y), pack_hi(v[2].y, v[3].y), pack_hi(v[4].y, v[5].y), pack_hi(v[6].y, v[7].y));
    } else {
        const uint2* v = R.v;
        const int r = (t % 16) * 4, kq = t / 16;  // k = 4 kq .. + 4: half kq % 2 of chunk kq / 2
        const int c = kq / 2, h = (kq % 2) * 4;
        *reinterpret_cast<uint2*>(S + lds_at(r + 0, c) + h) = make_uint2(pack_lo(v[0].x, v[1].x), pack_lo(v[2].x, v[3].x));
        *reinterpret_cast<uint2*>(S + lds_at(r + 1, c) + h) = make_uint2(pack_hi(v[0].x, v[1].x), pack_hi(v[2].x, v[3].x));
        *reinterpret_cast<uint2*>(S + lds_at(r + 2, c) + h) = make_uint2(pack_lo(v[0].y, v[1].y), pack_lo(v[2].y, v[3].y));
        *reinterpret_cast<uint2*>(S + lds_at(r + 3, c) + h) = make_uint2(pack_hi(v[0].y, v[1].y), pack_hi(v[2].y, v[3].y));
    }
}

// One BK-deep step of a wave's 64 x (32 NB) tile from the LDS operands.
template <int NB>
__device__ __forceinline__ void mma_tile(const __bf16* As, const __bf16* Bs, int wi, int wj, int lane,
                                         f32x16 (&acc)[2][NB]) {
#pragma unroll
    for (int ks = 0; ks < BK / 16; ks++) {
        const int c = ks * 2 + lane / 32;
        bf16x8 fa[2], fb[NB];
#pragma unroll
        for (int a = 0; a < 2; a++)
            fa[a] = *reinterpret_cast<const bf16x8*>(As + lds_at(wi + a * 32 + lane % 32, c));
#pragma unroll
        for (int b = 0; b < NB; b++)
            fb[b] = *reinterpret_cast<const bf16x8*>(Bs + lds_at(wj + b * 32 + lane % 32, c));
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int b = 0; b < NB; b++)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
}

// C[M,N] = A[M,K] B[K,N] (+ bias[N], then optionally GELU into act).
//  A_KCONT: A(i,k) = A[i*lda + k], else A[k*lda + i]
//  B_KCONT: B(k,j) = B[j*ldb + k], else B[k*ldb + j]
// A workgroup computes one 128 x BN tile (BN = 128 or 64) over the k range
// [z kchunk, (z + 1) kchunk); with work != NULL it writes that partial product
// to work[z] (row-major [M, N]) instead of the epilogue.  Four waves of 64 x 64,
// double-buffered LDS (one barrier per k tile), the next tile's global loads
// in flight during the matrix-core work on the current one.
// TA, TB: the operands' storage (float, rounded when staged, or __bf16);
// TACT: the storage of the GELU output.
// The operand tiles in LDS, and after the k loop the epilogue's staging tile.
template <int BN>
constexpr int gemm_smem_bytes() {
    return (2 * BM * BK + 2 * BN * BK) * (int)sizeof(__bf16);
}

// The k loop of one output tile: the XCD-aware tile of this workgroup
// (i0, j0, k part kz) and its accumulators.  Workgroups are dealt to the
// XCDs round-robin; they are renumbered so that each XCD takes one
// contiguous range of tiles (n fastest, then m, then the k part): its rows of
// A and the shared B stay in its own L2.
template <bool A_KCONT, bool B_KCONT, int BN, typename TA, typename TB>
__device__ __forceinline__ void gemm_mainloop(const TA* __restrict__ A, int lda, const TB* __restrict__ B, int ldb,
                                              int M, int N, int K, int kchunk, char* smem, int& i0, int& j0, int& kz,
                                              f32x16 (&acc)[2][BN / 64]) {
    constexpr int NB = BN / 64;  // 32-column MFMA tiles per wave
    __bf16 (*As)[BM * BK] = reinterpret_cast<__bf16 (*)[BM * BK]>(smem);
    __bf16 (*Bs)[BN * BK] = reinterpret_cast<__bf16 (*)[BN * BK]>(smem + 2 * BM * BK * sizeof(__bf16));
    const int nx = gridDim.x, ny = gridDim.y, nb = nx * ny * gridDim.z;
    const int bl = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
    const int q = nb / kXcd, rem = nb % kXcd, xcd = bl % kXcd;
    const int tile = xcd * q + min(xcd, rem) + bl / kXcd;
    i0 = (tile / nx) % ny * BM;
    j0 = tile % nx * BN;
    kz = tile / (nx * ny);
    const int kb = kz * kchunk, ke = min(K, kb + kchunk);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wi = (wave / 2) * 64, wj = (wave % 2) * (BN / 2);
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < NB; b++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[a][b][v] = 0.f;

    TileRegs<TA, A_KCONT, BM> ra;
    TileRegs<TB, B_KCONT, BN> rb;
    if (kb < ke) {
        load_tile<A_KCONT, BM>(A, lda, M, ke, i0, kb, ra);
        load_tile<B_KCONT, BN>(B, ldb, N, ke, j0, kb, rb);
        store_tile<A_KCONT, BM>(As[0], ra);
        store_tile<B_KCONT, BN>(Bs[0], rb);
    }
    __syncthreads();
    int cur = 0;
    for (int k0 = kb; k0 < ke; k0 += BK) {
        const bool more = k0 + BK < ke;
        if (more) {
            load_tile<A_KCONT, BM>(A, lda, M, ke, i0, k0 + BK, ra);
            load_tile<B_KCONT, BN>(B, ldb, N, ke, j0, k0 + BK, rb);
        }
        mma_tile<NB>(As[cur], Bs[cur], wi, wj, lane, acc);
        if (more) {  // the other buffer: every wave passed the last barrier after reading it
            store_tile<A_KCONT, BM>(As[cur ^ 1], ra);
            store_tile<B_KCONT, BN>(Bs[cur ^ 1], rb);
        }
        __syncthreads();
        cur ^= 1;
    }
}

template <bool A_KCONT, bool B_KCONT, int BN, typename TA, typename TB, typename TACT>
__global__ void __launch_bounds__(GEMM_THREADS) gemm_kernel(const TA* __restrict__ A, int lda,
                                                            const TB* __restrict__ B, int ldb, float* __restrict__ C,
                                                            int ldc, int M, int N, int K, int kchunk,
                                                            const float* __restrict__ bias, TACT* __restrict__ act,
                                                            int accumulate, float* __restrict__ work) {
    constexpr int NB = BN / 64;  // 32-column MFMA tiles per wave
    __shared__ __align__(16) char smem[gemm_smem_bytes<BN>()];
    int i0, j0, kz;
    f32x16 acc[2][NB];
    gemm_mainloop<A_KCONT, B_KCONT, BN>(A, lda, B, ldb, M, N, K, kchunk, smem, i0, j0, kz, acc);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wi = (wave / 2) * 64, wj = (wave % 2) * (BN / 2);
    // Lane holds column lane % 32 of each 32x32 tile, rows (v / 4) * 8 +
    // (lane / 32) * 4 + v % 4.
    // Epilogue through LDS, in two halves of 64 rows: the a = 0 (then
    // a = 1) accumulator tiles of every wave go to a row-major staging tile,
    // then each thread takes 4 consecutive columns of a row and stores them
    // as one 16-byte C vector (and one act vector), so that a wave writes
    // whole rows instead of 4-byte values (forward 4096 x 1024 x 1024: 27.6
    // -> 24.8 us).  The last k-loop barrier freed the operand tiles.
    if (work) {  // a split-K part: the raw partial product, stored directly (measured faster than staged)
        float* W = work + (size_t)kz * M * N;
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const int j = j0 + wj + b * 32 + lane % 32;
                if (j >= N) continue;
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const int i = i0 + wi + a * 32 + (v / 4) * 8 + (lane / 32) * 4 + v % 4;
                    if (i < M) W[(size_t)i * N + j] = acc[a][b][v];
                }
            }
        return;
    }
    constexpr int SROW = BN + 4;  // padded row stride of the staging tile (floats)
    constexpr int C4 = BN / 4;    // 4-column groups per row
    float* stage = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int a = 0; a < 2; a++) {
#pragma unroll
        for (int b = 0; b < NB; b++)
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const int lr = (wave / 2) * 32 + (v / 4) * 8 + (lane / 32) * 4 + v % 4;
                stage[lr * SROW + wj + b * 32 + lane % 32] = acc[a][b][v];
            }
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * C4; e += GEMM_THREADS) {
            const int lr = e / C4, c4 = e % C4;
            const int i = i0 + (lr / 32) * 64 + a * 32 + lr % 32;  // staging row -> output row
            const int j = j0 + c4 * 4;
            if (i >= M || j >= N) continue;
            float4 r = *reinterpret_cast<const float4*>(stage + lr * SROW + c4 * 4);
            if (bias) {
                r.x += bias[j];
                r.y += bias[j + 1];
                r.z += bias[j + 2];
                r.w += bias[j + 3];
            }
            if (C) {  // NULL: act is the only output (the host allows it without accumulate)
                float4* cp = reinterpret_cast<float4*>(C + (size_t)i * ldc + j);
                if (accumulate) {
                    const float4 c0 = *cp;
                    r.x += c0.x;
                    r.y += c0.y;
                    r.z += c0.z;
                    r.w += c0.w;
                }
                *cp = r;
            }
            if (act) {
                TACT* ap = act + (size_t)i * ldc + j;
                if constexpr (sizeof(TACT) == 2)
                    *reinterpret_cast<bf16x4*>(ap) = (bf16x4){to_bf16(gelu(r.x)), to_bf16(gelu(r.y)),
                                                              to_bf16(gelu(r.z)), to_bf16(gelu(r.w))};
                else
                    *reinterpret_cast<float4*>(ap) = make_float4(gelu(r.x), gelu(r.y), gelu(r.z), gelu(r.w));
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------- tiled products
// The products whose operands allow direct-to-LDS copies (tiled_operands):
// each BF16, or FP32 and k-contiguous.  See gemm_tile.h for the k loop.

// This workgroup's tile in an XCD-aware order (as gemm_mainloop's).
template <int BM, int BN>
__device__ __forceinline__ void xcd_tile(int& i0, int& j0, int& kz) {
    const int nx = gridDim.x, ny = gridDim.y, nb = nx * ny * gridDim.z;
    const int bl = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
    const int q = nb / kXcd, rem = nb % kXcd, xcd = bl % kXcd;
    const int tile = xcd * q + min(xcd, rem) + bl / kXcd;
    i0 = (tile / nx) % ny * BM;
    j0 = tile % nx * BN;
    kz = tile / (nx * ny);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Row-major staging of a workgroup's accumulators in LDS (rows SROW floats
// apart): lane holds column lane % 32 of each 32x32 tile, rows (v / 4) * 8 +
// (lane / 32) * 4 + v % 4.
template <int SROW, int NA, int NB>
__device__ __forceinline__ void stage_acc(float* stage, int wi, int wj, int lane,
                                          const f32x16 (&acc)[NA][NB]) {
#pragma unroll
    for (int a = 0; a < NA; a++)
#pragma unroll
        for (int b = 0; b < NB; b++)
#pragma unroll
            for (int v = 0; v < 16; v++)
                stage[(wi + a * 32 + (v / 4) * 8 + (lane / 32) * 4 + v % 4) * SROW + wj + b * 32 + lane % 32] =
                    acc[a][b][v];
}

template <class T, int BM, int BN>
constexpr int tile_smem_bytes() {  // the k loop's stages, then the epilogue's staging tile
    return T::kBytes > BM * (BN + 4) * 4 ? T::kBytes : BM * (BN + 4) * 4;
}

// C = A B with gemm_kernel's epilogues and arguments (act_bf16: act holds BF16).
template <typename TA, bool AK, typename TB, bool BK, int BM, int BN, int WM, int WN, int ST>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(1, 2)))
tile_gemm_kernel(const TA* __restrict__ A, int lda, const TB* __restrict__ B, int ldb, float* __restrict__ C, int ldc,
                 int M, int N, int K, int kchunk, const float* __restrict__ bias, void* __restrict__ act, int act_bf16,
                 int accumulate, float* __restrict__ work) {
    typedef tile::Tile<TA, AK, TB, BK, BM, BN, WM, WN, ST> T;
    __shared__ __align__(16) char smem[tile_smem_bytes<T, BM, BN>()];
    int i0, j0, kz;
    xcd_tile<BM, BN>(i0, j0, kz);
    const int kb = min(K, kz * kchunk), ke = min(K, kb + kchunk);
    f32x16 acc[T::NA][T::NB];
    T::run(A, lda, B, ldb, M, N, i0, j0, kb, ke, smem, acc);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wi = (wave / WN) * (BM / WM), wj = (wave % WN) * (BN / WN);
    if (work) {  // a split-K part: the raw partial product, stored directly
        float* W = work + (size_t)kz * M * N;
#pragma unroll
        for (int a = 0; a < T::NA; a++)
#pragma unroll
            for (int b = 0; b < T::NB; b++) {
                const int j = j0 + wj + b * 32 + lane % 32;
                if (j >= N) continue;
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const int i = i0 + wi + a * 32 + (v / 4) * 8 + (lane / 32) * 4 + v % 4;
                    if (i < M) W[(size_t)i * N + j] = acc[a][b][v];
                }
            }
        return;
    }
    constexpr int SROW = BN + 4, C4 = BN / 4, NT = 64 * WM * WN;
    float* stage = reinterpret_cast<float*>(smem);
    stage_acc<SROW>(stage, wi, wj, lane, acc);
    __syncthreads();
    const int c4 = threadIdx.x % C4, lr0 = threadIdx.x / C4, j = j0 + c4 * 4;  // a thread keeps its columns
    if (j >= N) return;
    f32x4 bv = {0.f, 0.f, 0.f, 0.f};
    if (bias) bv = (f32x4){bias[j], bias[j + 1], bias[j + 2], bias[j + 3]};
    // Beside an activation, C is the pre-activation that only a much later
    // backward reads: it is streamed past the caches (non-temporal).  The
    // outputs the next launch reads are not (the loss over a streamed z took
    // 96 us, over a cached one 87).
    auto rows = [&](auto to_c, auto act_kind) {  // act_kind: 0 none, 1 FP32, 2 BF16
        auto row = [&](int lr) {
            f32x4 r = *reinterpret_cast<const f32x4*>(stage + lr * SROW + c4 * 4);
            if (bias) r += bv;
            const size_t at = (size_t)(i0 + lr) * ldc + j;
            if constexpr (to_c.value) {
                f32x4* cp = reinterpret_cast<f32x4*>(C + at);
                if (accumulate) r += *cp;
                if constexpr (act_kind.value)
                    __builtin_nontemporal_store(r, cp);
                else
                    *cp = r;
            }
            if constexpr (act_kind.value == 2) {
                *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(act) + at) =
                    (bf16x4){to_bf16(gelu(r[0])), to_bf16(gelu(r[1])), to_bf16(gelu(r[2])), to_bf16(gelu(r[3]))};
            } else if constexpr (act_kind.value == 1) {
                *reinterpret_cast<f32x4*>(static_cast<float*>(act) + at) =
                    (f32x4){gelu(r[0]), gelu(r[1]), gelu(r[2]), gelu(r[3])};
            }
        };
        if (i0 + BM <= M) {
#pragma unroll 2
            for (int q = 0; q < BM * C4 / NT; q++) row(lr0 + q * (NT / C4));
        } else {
            for (int lr = lr0; i0 + lr < M; lr += NT / C4) row(lr);
        }
    };
    using std::integral_constant;
    if (!C)
        act_bf16 ? rows(std::false_type{}, integral_constant<int, 2>{}) : rows(std::false_type{}, integral_constant<int, 1>{});
    else if (!act)
        rows(std::true_type{}, integral_constant<int, 0>{});
    else
        act_bf16 ? rows(std::true_type{}, integral_constant<int, 2>{}) : rows(std::true_type{}, integral_constant<int, 1>{});
}

// gemm_gelu_bwd_kernel's product and epilogue on the tiled k loop: 128 rows
// (the column sums' blocks), BN columns.
template <typename TA, typename TB, int BN, int WM, int WN, int ST>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(1, 2)))
tile_gelu_bwd_kernel(const TA* __restrict__ A, int lda, const TB* __restrict__ B, int ldb,
                     const float* __restrict__ pre, int ldp, __bf16* __restrict__ out, int ldo, int M, int N, int K,
                     float* __restrict__ part) {
    typedef tile::Tile<TA, true, TB, false, BM, BN, WM, WN, ST> T;
    constexpr int SROW = BN + 4, C4 = BN / 4, NT = 64 * WM * WN, G = 4;
    static_assert(NT >= G * BN, "the column-sum groups");
    constexpr int kStageBytes = BM * SROW * 4, kTail = kStageBytes + G * BN * 4;
    __shared__ __align__(16) char smem[T::kBytes > kTail ? T::kBytes : kTail];
    float* stage = reinterpret_cast<float*>(smem);
    float (*sg)[BN] = reinterpret_cast<float (*)[BN]>(smem + kStageBytes);
    int i0, j0, kz;
    xcd_tile<BM, BN>(i0, j0, kz);
    f32x16 acc[T::NA][T::NB];
    T::run(A, lda, B, ldb, M, N, i0, j0, 0, K, smem, acc);
    // this thread's pre-activations (columns clamped to valid places, used inside N), in flight while the tile is
    // staged; rows past M are left out (4 x 512 x 64 5.5 -> 3.8 us) of a part tile only: the branches cost a whole
    // one 0.4 us
    constexpr int NR = BM * C4 / NT;
    const int c4 = threadIdx.x % C4, lr0 = threadIdx.x / C4, jc = j0 + c4 * 4, rows = min(BM, M - i0);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const float* pp = pre + min(jc, N - 4);
    auto epilogue = [&](auto whole) {
        float4 pr[NR];
#pragma unroll
        for (int q = 0; q < NR; q++)
            if (whole.value || lr0 + q * (NT / C4) < rows)
                pr[q] = *reinterpret_cast<const float4*>(pp + (size_t)(i0 + lr0 + q * (NT / C4)) * ldp);
        stage_acc<SROW>(stage, (wave / WN) * (BM / WM), (wave % WN) * (BN / WN), lane, acc);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NR; q++) {
            const int lr = lr0 + q * (NT / C4), i = i0 + lr;
            if (!whole.value && lr >= rows) continue;
            float4* sp = reinterpret_cast<float4*>(stage + lr * SROW + c4 * 4);
            const float4 dh = *sp;
            const float4 d = make_float4(dh.x * gelu_grad(pr[q].x), dh.y * gelu_grad(pr[q].y), dh.z * gelu_grad(pr[q].z),
                                         dh.w * gelu_grad(pr[q].w));
            if (jc < N)
                *reinterpret_cast<bf16x4*>(out + (size_t)i * ldo + jc) =
                    (bf16x4){to_bf16(d.x), to_bf16(d.y), to_bf16(d.z), to_bf16(d.w)};
            *sp = d;
        }
    };
    if (rows == BM)
        epilogue(std::true_type{});
    else
        epilogue(std::false_type{});
    __syncthreads();
    const int c = threadIdx.x % BN, g = threadIdx.x / BN, j = j0 + c;
    if (g < G) {
        float s = 0.f;
        if (rows == BM) {
#pragma unroll
            for (int r = 0; r < BM; r += G) s += stage[(g + r) * SROW + c];
        } else {
            for (int r = g; r < rows; r += G) s += stage[r * SROW + c];
        }
        sg[g][c] = s;
    }
    __syncthreads();
    if (g == 0 && j < N) part[(size_t)(i0 / BM) * N + j] = ((sg[0][c] + sg[1][c]) + sg[2][c]) + sg[3][c];
}

// dgrad with the GELU backward of the layer below in the epilogue (64-column
// tiles): d = (A B) * gelu'(pre), stored as BF16 (the operand rounding every
// later product applies anyway), and the column sums of each 128-row block of
// d in FP32 (the bias gradient's first pass), summed in the order of
// colsum_partial_kernel (rows g, g + 4, ... for g = 0..3, then the four
// groups in order), so the values equal the GEMM, gelu_bwd and colsum
// kernels in sequence bit for bit.
template <bool A_KCONT, bool B_KCONT, typename TA, typename TB>
__global__ void __launch_bounds__(GEMM_THREADS) gemm_gelu_bwd_kernel(const TA* __restrict__ A, int lda,
                                                                     const TB* __restrict__ B, int ldb,
                                                                     const float* __restrict__ pre, int ldp,
                                                                     __bf16* __restrict__ out, int ldo, int M, int N,
                                                                     int K, float* __restrict__ part) {
    constexpr int BN = 64, SROW = BN + 4, C4 = BN / 4;
    // the whole 128 x 64 FP32 tile (padded rows) and the column-sum groups fit the operand tiles' LDS
    static_assert(BM * SROW * 4 + 4 * 64 * 4 <= gemm_smem_bytes<BN>(), "staging tile");
    __shared__ __align__(16) char smem[gemm_smem_bytes<BN>()];
    int i0, j0, kz;
    f32x16 acc[2][1];
    gemm_mainloop<A_KCONT, B_KCONT, BN>(A, lda, B, ldb, M, N, K, K, smem, i0, j0, kz, acc);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wi = (wave / 2) * 64, wj = (wave % 2) * (BN / 2);
    float* stage = reinterpret_cast<float*>(smem);
    float (*sg)[64] = reinterpret_cast<float (*)[64]>(smem + BM * SROW * 4);
    // Lane holds column lane % 32 of each 32x32 tile, rows (v / 4) * 8 +
    // (lane / 32) * 4 + v % 4; the last k-loop barrier freed the operand tiles.
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int v = 0; v < 16; v++)
            stage[(wi + a * 32 + (v / 4) * 8 + (lane / 32) * 4 + v % 4) * SROW + wj + lane % 32] = acc[a][0][v];
    __syncthreads();
    for (int e = threadIdx.x; e < BM * C4; e += GEMM_THREADS) {
        const int lr = e / C4, c4 = e % C4;
        const int i = i0 + lr, j = j0 + c4 * 4;
        if (i >= M || j >= N) continue;
        float4* sp = reinterpret_cast<float4*>(stage + lr * SROW + c4 * 4);
        const float4 dh = *sp;
        const float4 pr = *reinterpret_cast<const float4*>(pre + (size_t)i * ldp + j);
        const float4 d = make_float4(dh.x * gelu_grad(pr.x), dh.y * gelu_grad(pr.y), dh.z * gelu_grad(pr.z),
                                     dh.w * gelu_grad(pr.w));
        *reinterpret_cast<bf16x4*>(out + (size_t)i * ldo + j) =
            (bf16x4){to_bf16(d.x), to_bf16(d.y), to_bf16(d.z), to_bf16(d.w)};
        *sp = d;
    }
    __syncthreads();
    const int c = threadIdx.x % 64, g = threadIdx.x / 64, j = j0 + c;
    const int rows = min(BM, M - i0);
    float s = 0.f;
    if (j < N)
        for (int r = g; r < rows; r += 4) s += stage[r * SROW + c];
    sg[g][c] = s;
    __syncthreads();
    if (g == 0 && j < N) part[(size_t)(i0 / BM) * N + j] = ((sg[0][c] + sg[1][c]) + sg[2][c]) + sg[3][c];
}

// Split-K epilogue: C = sum over the parts in order (part 0 first) + bias
// (+ C when accumulating), GELU into act; four columns per thread.
template <typename TACT>
__global__ void splitk_sum_kernel(const float* __restrict__ work, int splits, int M, int N, float* __restrict__ C,
                                  int ldc, const float* __restrict__ bias, TACT* __restrict__ act, int accumulate) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int n4 = N / 4;
    if (idx >= (int64_t)M * n4) return;
    const int i = (int)(idx / n4), j = (int)(idx % n4) * 4;
    const size_t mn = (size_t)M * N;
    const float* w = work + (size_t)i * N + j;
    float4 s = *reinterpret_cast<const float4*>(w);
    for (int z = 1; z < splits; z++) {
        const float4 t = *reinterpret_cast<const float4*>(w + z * mn);
        s.x += t.x;
        s.y += t.y;
        s.z += t.z;
        s.w += t.w;
    }
    if (bias) {
        s.x += bias[j];
        s.y += bias[j + 1];
        s.z += bias[j + 2];
        s.w += bias[j + 3];
    }
    float4* cp = reinterpret_cast<float4*>(C + (size_t)i * ldc + j);
    if (accumulate) {
        const float4 c = *cp;
        s.x += c.x;
        s.y += c.y;
        s.z += c.z;
        s.w += c.w;
    }
    *cp = s;
    if (act) {
        TACT* ap = act + (size_t)i * ldc + j;
        ap[0] = (TACT)gelu(s.x);
        ap[1] = (TACT)gelu(s.y);
        ap[2] = (TACT)gelu(s.z);
        ap[3] = (TACT)gelu(s.w);
    }
}

__global__ void gelu_bwd_kernel(const float* __restrict__ pre, const float* __restrict__ dact,
                                float* __restrict__ dpre, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dpre[i] = dact[i] * gelu_grad(pre[i]);
}

// Column sums of a row-major [M, N] matrix, deterministic.  Pass 1: per
// 128-row chunk and 64-column stripe, four row groups (rows g, g + 4, ...)
// each sum in row order, then the four groups in order.  Pass 2: the chunk
// sums of each column the same way (chunks g, g + 4, ..., then the groups).
constexpr int COLSUM_ROWS = 128;
// Xb (may be NULL): X rounded to BF16, on the way.  next (may be NULL):
// receives *step + 1, for a later launch to read.
__global__ void __launch_bounds__(256) colsum_partial_kernel(const float* __restrict__ X, int M, int N,
                                                             float* __restrict__ part, __bf16* __restrict__ Xb,
                                                             const int32_t* __restrict__ step,
                                                             int32_t* __restrict__ next) {
    if (next && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *next = *step + 1;
    __shared__ float s[4][64];
    const int c = threadIdx.x % 64, g = threadIdx.x / 64;
    const int j = blockIdx.x * 64 + c;
    const int i0 = blockIdx.y * COLSUM_ROWS, i1 = min(i0 + COLSUM_ROWS, M);
    float acc = 0.f;
    if (j < N) {
        int i = i0 + g;
        for (; i + 28 < i1; i += 32) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) v[u] = X[(size_t)(i + 4 * u) * N + j];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                acc += v[u];
                if (Xb) Xb[(size_t)(i + 4 * u) * N + j] = to_bf16(v[u]);
            }
        }
        for (; i < i1; i += 4) {
            const float v = X[(size_t)i * N + j];
            acc += v;
            if (Xb) Xb[(size_t)i * N + j] = to_bf16(v);
        }
    }
    s[g][c] = acc;
    __syncthreads();
    if (g == 0 && j < N) part[(size_t)blockIdx.y * N + j] = ((s[0][c] + s[1][c]) + s[2][c]) + s[3][c];
}
__global__ void __launch_bounds__(256) colsum_final_kernel(const float* __restrict__ part, int chunks, int N,
                                                           float* __restrict__ out, float scale) {
    __shared__ float s[4][64];
    const int c = threadIdx.x % 64, g = threadIdx.x / 64;
    const int j = blockIdx.x * 64 + c;
    float acc = 0.f;
    if (j < N)
        for (int k = g; k < chunks; k += 4) acc += part[(size_t)k * N + j];
    s[g][c] = acc;
    __syncthreads();
    if (g == 0 && j < N) out[j] = (((s[0][c] + s[1][c]) + s[2][c]) + s[3][c]) * scale;
}

// Adam (Kingma and Ba, 2015) with bias correction; FP32 state.
// pb (may be NULL) receives the updated parameters rounded to BF16: the
// matrix cores' copy of the weights.
// One parameter's Adam update (Kingma and Ba, Algorithm 1, with the bias
// corrections c1, c2).  No contraction, so that every kernel below rounds
// each operation alike whatever the compiler would fuse in its context.
__device__ __forceinline__ void adam_one(float& p, float g, float& m1, float& m2, float lr, float b1, float b2,
                                         float eps, float c1, float c2) {
#pragma clang fp contract(off)
    const float a = b1 * m1 + (1.f - b1) * g;
    const float b = b2 * m2 + (1.f - b2) * g * g;
    m1 = a;
    m2 = b;
    p = p - lr * (a / c1) / (sqrtf(b / c2) + eps);
}

__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m1,
                            float* __restrict__ m2, int64_t n, float lr, float b1, float b2, float eps, float c1,
                            float c2, __bf16* __restrict__ pb) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float pi = p[i], ai = m1[i], bi = m2[i];
    adam_one(pi, g[i], ai, bi, lr, b1, b2, eps, c1, c2);
    m1[i] = ai;
    m2[i] = bi;
    p[i] = pi;
    if (pb) pb[i] = to_bf16(pi);
}

// Adam with the step count in device memory (a recorded step replays with
// the count it finds there): each workgroup forms the bias corrections from
// step + 1, and step_bump_kernel, launched after it, stores step + 1.
__global__ void adam_dev_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m1,
                                float* __restrict__ m2, int64_t n, float lr, float b1, float b2, float eps,
                                const int32_t* __restrict__ step, __bf16* __restrict__ pb) {
    __shared__ float corr[2];  // the bias corrections, formed once per workgroup
    if (threadIdx.x == 0) {
        const float t = (float)(*step + 1);
        corr[0] = 1.f - powf(b1, t);
        corr[1] = 1.f - powf(b2, t);
    }
    __syncthreads();
    const float c1 = corr[0], c2 = corr[1];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float pi = p[i], ai = m1[i], bi = m2[i];
    adam_one(pi, g[i], ai, bi, lr, b1, b2, eps, c1, c2);
    m1[i] = ai;
    m2[i] = bi;
    p[i] = pi;
    if (pb) pb[i] = to_bf16(pi);
}

// adam_dev_kernel over 4 consecutive parameters per thread (16-byte
// accesses) in a grid-stride loop: the same arithmetic per parameter, the
// bias corrections formed once per workgroup for many more parameters.
__global__ void __launch_bounds__(256) adam_dev4_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                        float* __restrict__ m1, float* __restrict__ m2, int64_t n,
                                                        float lr, float b1, float b2, float eps,
                                                        const int32_t* __restrict__ step, __bf16* __restrict__ pb) {
    __shared__ float corr[2];
    if (threadIdx.x == 0) {
        const float t = (float)(*step + 1);
        corr[0] = 1.f - powf(b1, t);
        corr[1] = 1.f - powf(b2, t);
    }
    __syncthreads();
    const float c1 = corr[0], c2 = corr[1];
    const int64_t n4 = n / 4, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n4; q += stride) {
        float4 pv = reinterpret_cast<float4*>(p)[q];
        float4 av = reinterpret_cast<float4*>(m1)[q];
        float4 bv = reinterpret_cast<float4*>(m2)[q];
        const float4 gv = reinterpret_cast<const float4*>(g)[q];
        adam_one(pv.x, gv.x, av.x, bv.x, lr, b1, b2, eps, c1, c2);
        adam_one(pv.y, gv.y, av.y, bv.y, lr, b1, b2, eps, c1, c2);
        adam_one(pv.z, gv.z, av.z, bv.z, lr, b1, b2, eps, c1, c2);
        adam_one(pv.w, gv.w, av.w, bv.w, lr, b1, b2, eps, c1, c2);
        reinterpret_cast<float4*>(m1)[q] = av;
        reinterpret_cast<float4*>(m2)[q] = bv;
        reinterpret_cast<float4*>(p)[q] = pv;
        if (pb)
            reinterpret_cast<bf16x4*>(pb)[q] = (bf16x4){to_bf16(pv.x), to_bf16(pv.y), to_bf16(pv.z), to_bf16(pv.w)};
    }
    for (int64_t i = 4 * n4 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        float pi = p[i], ai = m1[i], bi = m2[i];
        adam_one(pi, g[i], ai, bi, lr, b1, b2, eps, c1, c2);
        m1[i] = ai;
        m2[i] = bi;
        p[i] = pi;
        if (pb) pb[i] = to_bf16(pi);
    }
}

// The training step's gradients and Adam in one pass over the parameters of
// up to kUpdateLayers layers: each thread sums four weights' split-K parts in
// part order (splitk_sum_kernel's sum) and updates them; the blocks after the
// weights' form 64 bias gradients each (colsum_final_kernel's second pass) and
// update those.  Bound by memory: per weight 4 bytes of each part, 24 of
// parameter and moments, 2 of the BF16 copy.  The gradient itself never
// reaches memory, and one launch replaces a sum per layer, Adam and the step
// count's own (4,096-sample step on one card, in turn: 348 -> 334 us; this kernel 31 us for 145 MB).  This step's count is the
// one that its column-sum pass left in the scratch; the launch that has step
// stores it there, so a step that fails before its update leaves Adam's count
// as it was.  VEC: 16-byte accesses of parameters and moments.
template <bool VEC>
__device__ __forceinline__ float4 load4(const float* p) {
    if constexpr (VEC)
        return *reinterpret_cast<const float4*>(p);
    else
        return make_float4(p[0], p[1], p[2], p[3]);
}
template <bool VEC>
__device__ __forceinline__ void store4(float* p, const float4& v) {
    if constexpr (VEC) {
        *reinterpret_cast<float4*>(p) = v;
    } else {
        p[0] = v.x;
        p[1] = v.y;
        p[2] = v.z;
        p[3] = v.w;
    }
}
template <bool VEC>
__global__ void __launch_bounds__(256) update_kernel(UpdateLayers u, float* __restrict__ p, float* __restrict__ m1,
                                                     float* __restrict__ m2, __bf16* __restrict__ pb, float lr,
                                                     float b1, float b2, float eps,
                                                     const int32_t* __restrict__ count, int32_t* __restrict__ step) {
    __shared__ float corr[2], sg[4][64];
    const int blk = blockIdx.x;
    int k = 0;
    while (k + 1 < u.n && blk >= u.layer[k + 1].first) k++;
    const UpdateLayer& L = u.layer[k];
    if (threadIdx.x == 0) {
        const int32_t n = *count;
        if (step && blk == 0) *step = n;
        const float t = (float)n;
        corr[0] = 1.f - powf(b1, t);
        corr[1] = 1.f - powf(b2, t);
    }
    if (blk < L.first + L.weight_blocks) {
        const int64_t n4 = (int64_t)L.fo * L.fi / 4, q = (int64_t)(blk - L.first) * 256 + threadIdx.x;
        const bool in = q < n4;
        float4 pv, av, bv, g;
        const int64_t at = L.wo + 4 * q;
        if (in) {  // every load ahead of the barrier
            pv = load4<VEC>(p + at);
            av = load4<VEC>(m1 + at);
            bv = load4<VEC>(m2 + at);
            g = *reinterpret_cast<const float4*>(L.work + 4 * q);
            for (int z = 1; z < L.splits; z++) {
                const float4 t = *reinterpret_cast<const float4*>(L.work + 4 * q + z * 4 * n4);
                g.x += t.x;
                g.y += t.y;
                g.z += t.z;
                g.w += t.w;
            }
        }
        __syncthreads();
        if (!in) return;
        const float c1 = corr[0], c2 = corr[1];
        adam_one(pv.x, g.x, av.x, bv.x, lr, b1, b2, eps, c1, c2);
        adam_one(pv.y, g.y, av.y, bv.y, lr, b1, b2, eps, c1, c2);
        adam_one(pv.z, g.z, av.z, bv.z, lr, b1, b2, eps, c1, c2);
        adam_one(pv.w, g.w, av.w, bv.w, lr, b1, b2, eps, c1, c2);
        store4<VEC>(m1 + at, av);
        store4<VEC>(m2 + at, bv);
        store4<VEC>(p + at, pv);
        if (pb)
            *reinterpret_cast<bf16x4*>(pb + at) = (bf16x4){to_bf16(pv.x), to_bf16(pv.y), to_bf16(pv.z), to_bf16(pv.w)};
        return;
    }
    const int c = threadIdx.x % 64, g = threadIdx.x / 64;
    const int j = (blk - L.first - L.weight_blocks) * 64 + c;
    float acc = 0.f;
    if (j < L.fo)
        for (int z = g; z < u.chunks; z += 4) acc += L.part[(size_t)z * L.fo + j];
    sg[g][c] = acc;
    __syncthreads();
    if (g == 0 && j < L.fo) {
        const int64_t at = L.wo + (int64_t)L.fo * L.fi + j;
        float pi = p[at], ai = m1[at], bi = m2[at];
        adam_one(pi, (((sg[0][c] + sg[1][c]) + sg[2][c]) + sg[3][c]) * 1.0f, ai, bi, lr, b1, b2, eps, corr[0], corr[1]);
        m1[at] = ai;
        m2[at] = bi;
        p[at] = pi;
        if (pb) pb[at] = to_bf16(pi);
    }
}

__global__ void step_bump_kernel(int32_t* step) { *step += 1; }

__global__ void to_bf16_kernel(const float* __restrict__ x, int64_t n, __bf16* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = to_bf16(x[i]);
}

__global__ void __launch_bounds__(256) to_bf16x8_kernel(const float* __restrict__ x, int64_t n8,
                                                        __bf16* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n8) return;
    const float4 a = reinterpret_cast<const float4*>(x)[2 * i], b = reinterpret_cast<const float4*>(x)[2 * i + 1];
    reinterpret_cast<bf16x8*>(y)[i] = pack8(a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w);
}

// p[i] from a uniform base and a 32-bit byte offset (one address instruction
// instead of a 64-bit sum per lane; the arrays are far below 4 GiB).
template <typename T>
__device__ __forceinline__ T at(const T* p, uint32_t i) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + i * (uint32_t)sizeof(T));
}

__device__ __forceinline__ double sigmoid(double z) { return 1.0 / (1.0 + exp(-z)); }

// Entry e < 2N + 2G (va, vm, pg, qg blocks of x) of the squashed network
// output zb (vm, va, pg, qg blocks, FP32), and in act the activation it
// came from (tanh for va, the sigmoid otherwise): the squashing kernel and
// the fused loss kernel both call it, so both write the same bits.
__device__ __forceinline__ double squash_entry(const ProxBox& box, const float* zb, int e, double& act) {
    const int N = box.N, G = box.G;
    if (e < N) {  // va
        act = tanh((double)at(zb, N + e));
        return at(box.is_ref, e) ? 0.0 : box.va_span * act;
    }
    if (e < 2 * N) {  // vm
        const int i = e - N;
        act = sigmoid((double)at(zb, i));
        return at(box.vmin, i) + (at(box.vmax, i) - at(box.vmin, i)) * act;
    }
    if (e < 2 * N + G) {
        const int k = e - 2 * N;
        act = sigmoid((double)at(zb, 2 * N + k));
        return at(box.pmin, k) + (at(box.pmax, k) - at(box.pmin, k)) * act;
    }
    const int k = e - 2 * N - G;
    act = sigmoid((double)at(zb, 2 * N + G + k));
    return at(box.qmin, k) + (at(box.qmax, k) - at(box.qmin, k)) * act;
}

// z [B, 2N + 2G] (vm, va, pg, qg blocks, FP32) -> the first 2N + 2G entries
// of each instance's x [B, n] (va, vm, pg, qg, FP64); p and q are zeroed.
// per = n writes every entry (p, q = 0); per = 2N + 2G leaves p, q as they are.
__global__ void squash_fwd_kernel(const float* __restrict__ z, int B, ProxBox box, double* __restrict__ X,
                                  int64_t n, int64_t per) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int D = 2 * box.N + 2 * box.G;
    if (idx >= (int64_t)B * per) return;
    const int64_t b = idx / per;
    const int64_t e = idx % per;
    double act;
    X[b * n + e] = e < D ? squash_entry(box, z + b * D, (int)e, act) : 0.0;
}

// dz from dL/dx = gX + gX2 + obj_scale * gObj on the (va, vm, pg, qg)
// entries (gX2, gObj may be NULL).
__global__ void squash_bwd_kernel(const float* __restrict__ z, int B, ProxBox box, const double* __restrict__ gX1,
                                  const double* __restrict__ gX2, const double* __restrict__ gObj, double obj_scale,
                                  int64_t n, float* __restrict__ dz, float scale) {
    const int D = 2 * box.N + 2 * box.G;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)B * D) return;
    const int64_t b = idx / D;
    const int j = (int)(idx % D);
    const int N = box.N, G = box.G;
    const double zj = z[idx];
    // the x entry this output feeds
    int64_t e;
    if (j < N) e = N + j;                    // vm
    else if (j < 2 * N) e = j - N;           // va
    else e = j;                              // pg, qg: same offset in z and x
    double g = gX1[b * n + e];
    if (gX2) g += gX2[b * n + e];
    if (gObj) g += obj_scale * gObj[b * n + e];
    double d;
    if (j < N) {  // vm
        const double s = sigmoid(zj);
        d = g * (box.vmax[j] - box.vmin[j]) * s * (1.0 - s);
    } else if (j < 2 * N) {  // va
        const int i = j - N;
        const double t = tanh(zj);
        d = box.is_ref[i] ? 0.0 : g * box.va_span * (1.0 - t * t);
    } else if (j < 2 * N + G) {
        const int k = j - 2 * N;
        const double s = sigmoid(zj);
        d = g * (box.pmax[k] - box.pmin[k]) * s * (1.0 - s);
    } else {
        const int k = j - 2 * N - G;
        const double s = sigmoid(zj);
        d = g * (box.qmax[k] - box.qmin[k]) * s * (1.0 - s);
    }
    dz[idx] = (float)(d * scale);
}

// dz = (d x / d z)^T g with g = wb[b] (gX1 + obj_scale grad f(X)) on the
// va, vm, pg, qg entries (grad f = 2 c2 pg + c1 on pg): the objective and
// loss-weight step of vjp_sum_kernel and squash_bwd_kernel in one pass, in
// the same order of operations.
__global__ void loss_bwd_kernel(const float* __restrict__ z, int B, ProxBox box, ProxObj ob,
                                const double* __restrict__ X, const double* __restrict__ gX1, double obj_scale,
                                const double* __restrict__ wb, int64_t n, float* __restrict__ dz) {
    const int D = 2 * box.N + 2 * box.G;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)B * D) return;
    const int64_t b = idx / D;
    const int j = (int)(idx % D);
    const int N = box.N, G = box.G;
    const double zj = z[idx];
    int64_t e;
    if (j < N) e = N + j;                    // vm
    else if (j < 2 * N) e = j - N;           // va
    else e = j;                              // pg, qg: same offset in z and x
    double g = gX1[b * n + e];
    if (X && j >= 2 * N && j < 2 * N + G) {
        const int k = j - 2 * N;
        g += obj_scale * (2.0 * ob.c2[k] * X[b * n + e] + ob.c1[k]);
    }
    g *= wb[b];
    double d;
    if (j < N) {  // vm
        const double s = sigmoid(zj);
        d = g * (box.vmax[j] - box.vmin[j]) * s * (1.0 - s);
    } else if (j < 2 * N) {  // va
        const int i = j - N;
        const double t = tanh(zj);
        d = box.is_ref[i] ? 0.0 : g * box.va_span * (1.0 - t * t);
    } else if (j < 2 * N + G) {
        const int k = j - 2 * N;
        const double s = sigmoid(zj);
        d = g * (box.pmax[k] - box.pmin[k]) * s * (1.0 - s);
    } else {
        const int k = j - 2 * N - G;
        const double s = sigmoid(zj);
        d = g * (box.qmax[k] - box.qmin[k]) * s * (1.0 - s);
    }
    dz[idx] = (float)d;
}

// The arc flows p, q are F(vm, va): a gradient on them reaches the
// voltages through the flow rows c = p - F, whose va / vm columns are -dF.
// With G1 = J^T W, the arc entry of the total gradient is G1 + gpq, and
// J^T W2 with w2 = -(G1 + gpq) on the arc's flow row carries it to va, vm.
// G1 has a closed form on the arc variables: column p_a of J holds the flow
// row (weight 0 in W), the branch side's thermal row (2 p_a) and the active
// balance row of the arc's bus (1); q_a likewise with the reactive row.  So
// the total weights Wt = W + W2 need no first product, and the VJP is the
// single product J^T Wt.  w2 of flow row rr (0 .. 4L) of one instance:
__device__ __forceinline__ double flow_weight(const double* x, const double* w, const double* gq, const ProxRows& rows,
                                              int rr) {
    // flow rows p_fr[L], q_fr[L], p_to[L], q_to[L]
    const int L = rows.L;
    const int blk = rr / L, l = rr % L;
    const bool from = blk == 0 || blk == 1, isq = blk == 1 || blk == 3;
    const int q = (isq ? 2 * L : 0) + (from ? l : L + l);  // index inside the p, q entries
    const int bus = from ? rows.f_bus[l] : rows.t_bus[l];
    const double g1 = 2.0 * x[rows.pq0 + q] * w[(from ? rows.thf : rows.tht) + l] + w[(isq ? rows.balq : rows.balp) + bus];
    return -(g1 + gq[q]);
}

// The wave's sums of N values (a power of two) at once: lane q * 64 / N
// receives value q's, each added in the tree of shuffles by 32, 16, .. 1 (the
// first steps halve the values instead of repeating them for each); and the
// largest mx beside them, in lane 0.
template <int N>
__device__ __forceinline__ double wave_sums(const double (&v)[N], double& mx) {
    const int lane = threadIdx.x & 63;
    double a[N];
#pragma unroll
    for (int q = 0; q < N; q++) a[q] = v[q];
#pragma unroll
    for (int s = 32; s > 0; s /= 2) {
        const int n = N * s / 64;  // values that stay in a lane
        if (n > 0) {
            const bool up = lane & s;
#pragma unroll
            for (int q = 0; q < n; q++) {
                const double keep = up ? a[q + n] : a[q], send = up ? a[q] : a[q + n];
                a[q] = keep + __shfl_xor(send, s, 64);
            }
        } else {
            a[0] += __shfl_down(a[0], s, 64);
        }
        mx = fmax(mx, __shfl_down(mx, s, 64));
    }
    return a[0];
}

// Per instance b: the loss rho * (sum over non-flow rows of viol^2 + sum
// over p, q of bound viol^2) + obj_scale * F[b] (F may be NULL), the
// constraint violation (max over all rows and variable bounds), the weights
// w = d penalty / d c (zero on flow rows) and d penalty / d x on the p, q
// entries.  One workgroup of NT threads per instance.  The sum runs in LANES
// lanes (row r in lane r % LANES, rows ascending), then over the lanes of each
// 64 in shuffle order, then over those in order; a thread holds the lanes
// LANES / NT apart, so a sample's loss is the same bits whichever NT its
// batch takes.
// Bound by the latency of its loads: a thread's loop holds kPenRows rows'
// loads in flight, and few instances of many rows take more threads each (256
// instances of 1,000 buses, 70 MB: 57.2 us with 256 threads and one row at a
// time, 33.5 us with four rows, 18.6 us with 1,024 threads as well).
constexpr int kPenRows = 4;
template <int NT, int LANES>
__global__ void __launch_bounds__(NT) penalty_kernel(const double* __restrict__ C, const double* __restrict__ X,
                                                     const double* __restrict__ F, double obj_scale, ProxRows rows,
                                                     double rho, double* __restrict__ pen, double* __restrict__ cvio,
                                                     double* W, double* gpq, int vjp) {
    constexpr int U = LANES / NT;
    static_assert(kPenRows % U == 0, "a thread's rows in flight cover its lanes");
    __shared__ double s_pen[LANES / 64], s_vio[NT / 64];
    extern __shared__ double s_gq[];  // d pen / d (p, q) when gpq is NULL (vjp only)
    const int64_t b = blockIdx.x;
    const double* c = C + b * rows.m;
    const double* x = X + b * rows.n;
    double* w = W + b * rows.m;
    double* gq = gpq ? gpq + b * rows.npq : s_gq;
    double sp[U] = {}, sv = 0.0;
    auto viol_of = [](double v, double lo, double hi) { return v < lo ? v - lo : (v > hi ? v - hi : 0.0); };
    auto each = [&](int count, auto load, auto use) {  // load(u, r) of kPenRows rows, then use(u, r)
        int r = threadIdx.x;
        for (; r + (kPenRows - 1) * NT < count; r += kPenRows * NT) {
#pragma unroll
            for (int u = 0; u < kPenRows; u++) load(u, r + u * NT);
#pragma unroll
            for (int u = 0; u < kPenRows; u++) use(u, r + u * NT);
        }
        if constexpr (U == 1) {
            for (; r < count; r += NT) {
                load(0, r);
                use(0, r);
            }
        } else {
#pragma unroll
            for (int u = 0; u < kPenRows - 1; u++) {
                if (r + u * NT >= count) break;
                load(u, r + u * NT);
                use(u, r + u * NT);
            }
        }
    };
    double v[kPenRows], lo[kPenRows], hi[kPenRows];
    each(
        rows.m,
        [&](int u, int r) {
            v[u] = c[r];
            lo[u] = rows.lcon[r];
            hi[u] = rows.ucon[r];
        },
        [&](int u, int r) {
            const double dv = viol_of(v[u], lo[u], hi[u]);
            sv = fmax(sv, fabs(dv));
            const bool flow = r >= rows.flow0 && r < rows.flow1;
            if (!flow) sp[u % U] = fma(dv, dv, sp[u % U]);
            if (!(flow && vjp)) w[r] = flow ? 0.0 : 2.0 * rho * dv;  // with vjp the flow rows come below
        });
    each(
        rows.npq,
        [&](int u, int q) {
            v[u] = x[rows.pq0 + q];
            lo[u] = rows.lvar[rows.pq0 + q];
            hi[u] = rows.uvar[rows.pq0 + q];
        },
        [&](int u, int q) {
            const double dv = viol_of(v[u], lo[u], hi[u]);
            sv = fmax(sv, fabs(dv));
            sp[u % U] = fma(dv, dv, sp[u % U]);
            gq[q] = 2.0 * rho * dv;
        });
    const double sum = wave_sums(sp, sv);
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    if (lane % (64 / U) == 0) s_pen[lane / (64 / U) * (NT / 64) + wave] = sum;
    if (lane == 0) s_vio[wave] = sv;
    __syncthreads();
    if (threadIdx.x == 0) {
        double P = 0.0, V = 0.0;
        for (int q = 0; q < LANES / 64; q++) P += s_pen[q];
        for (int q = 0; q < NT / 64; q++) V = fmax(V, s_vio[q]);
        pen[b] = F ? rho * P + obj_scale * F[b] : rho * P;
        cvio[b] = V;
    }
    if (vjp) {  // the workgroup's W and gpq stores are visible after the barrier above
        for (int rr = threadIdx.x; rr < rows.flow1 - rows.flow0; rr += NT)
            w[rows.flow0 + rr] = flow_weight(x, w, gq, rows, rr);
    }
}

// The VJP weights on their own (prox_vjp_weights): one thread per flow row.
// The flow rows of Wt are written from W's thermal and balance rows, which
// they never overlap, so Wt may be W itself; a separate Wt also receives W's
// other rows.
__global__ void vjp_weights_kernel(const double* X, const double* W, const double* __restrict__ gpq, ProxRows rows,
                                   int B, double* Wt) {
    const int nf = rows.flow1 - rows.flow0;  // 4 L
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)B * nf) return;
    const int64_t b = idx / nf;
    const int rr = (int)(idx % nf);
    Wt[b * rows.m + rows.flow0 + rr] = flow_weight(X + b * rows.n, W + b * rows.m, gpq + b * rows.npq, rows, rr);
}
__global__ void copy_off_flow_kernel(const double* __restrict__ W, ProxRows rows, int B, double* __restrict__ Wt) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)B * rows.m) return;
    const int r = (int)(idx % rows.m);
    if (r < rows.flow0 || r >= rows.flow1) Wt[idx] = W[idx];
}

// gX [B, n] = wb[b] * (gX1 + gX2 + obj_scale * grad f) on the va, vm, pg, qg
// entries (the free variables of the proxy), zero on the arc variables;
// grad f = 2 c2 pg + c1 on the pg entries, 0 elsewhere (static model).
__global__ void vjp_sum_kernel(const double* __restrict__ X, const double* __restrict__ gX1,
                               const double* __restrict__ gX2, ProxObj ob, double obj_scale,
                               const double* __restrict__ wb, int B, int64_t n, int64_t nfree,
                               double* __restrict__ gX) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)B * n) return;
    const int64_t b = idx / n, e = idx % n;
    double g = 0.0;
    if (e < nfree) {
        g = gX1[idx];
        if (gX2) g += gX2[idx];
        if (X && e >= ob.x_pg && e < ob.x_pg + ob.G) {
            const int64_t k = e - ob.x_pg;
            g += obj_scale * (2.0 * ob.c2[k] * X[idx] + ob.c1[k]);
        }
        g *= wb[b];
    }
    gX[idx] = g;
}

// The proxy's training samples from uniform draws r [B, N] in [0, 1): bus
// i's pd and qd both scaled by 1 + spread (2 r - 1); loads [B, 2N] (pd then
// qd) and the network's features (loads - base) * inv_scale as FP32.  The
// operations of the host formula one by one, uncontracted.
__global__ void sample_loads_kernel(const double* __restrict__ r, const double* __restrict__ base,
                                    const double* __restrict__ inv_scale, double spread, int B, int N,
                                    double* __restrict__ loads, float* __restrict__ feats) {
#pragma clang fp contract(off)
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t tot = (int64_t)B * 2 * N;
    if (idx >= tot) return;
    const int64_t b = idx / (2 * N);
    const int j = (int)(idx % (2 * N)), i = j < N ? j : j - N;
    const double u = r[b * N + i] * 2.0 - 1.0;
    const double fac = 1.0 + spread * u;
    const double l = base[j] * fac;
    loads[idx] = l;
    feats[idx] = (float)((l - base[j]) * inv_scale[j]);
}

// ------------------------------------------------------------ fused loss
// The whole FP64 side of the training loss in one launch, one workgroup per
// sample, every intermediate in LDS: squashing, the arc flows p, q := F(vm,
// va), the non-flow rows (reference, angle, balance, thermal), the penalty,
// the largest violation and, when asked, d loss / d z.  Only z, the loads
// and the model's read-only arrays are read, and only the loss, Cvio and
// d loss / d z are written (X and C on request): about 14 KB per 300-bus
// sample, where the chain of batch launches moves [B, n] and [B, m] arrays
// through HBM several times.
//
// The gradient is the same chain as the penalty VJP (J^T of the row
// weights, carried to the voltages through the flows), written per branch
// and summed per bus over the bus's half-edges in adjacency order (no
// atomics: the same bits on every run).
//
// Flow, thermal-row and objective-term arithmetic is not contracted, as in
// the callback kernels, so the arc flows, thermal rows and X equal those of
// the batch launches bit for bit; the per-bus and per-sample sums are
// ordered differently (rounding-level differences in the balance rows, the
// loss and the gradient).
// F = al u^2 + be w^2 + u w (a C + b S) and its derivatives in u, w and the
// angle difference (the expression of the callback kernels' flow terms).
struct PFlow {
    double F, Fu, Fw, Ft;
};
__device__ __forceinline__ PFlow pflow(double al, double be, double a, double b, double u, double w, double C,
                                       double S) {
#pragma clang fp contract(off)
    const double k1 = a * C + b * S;
    const double k2 = b * C - a * S;
    const double uw = u * w;
    PFlow r;
    r.F = al * u * u + be * w * w + uw * k1;
    r.Fu = 2.0 * al * u + w * k1;
    r.Fw = 2.0 * be * w + u * k1;
    r.Ft = uw * k2;
    return r;
}

__device__ __forceinline__ double viol(double v, double lo, double hi) {
    return v < lo ? v - lo : (v > hi ? v - hi : 0.0);
}

// Branch l's packed values (ProxPerm::br).
struct BranchCoef {
    double2 ff, ft, tt, tf;  // (G, B) of each side pair
};
__device__ __forceinline__ double2 branch_pair(const double2* br, int L, int k, uint32_t l) {
    return at(br + (size_t)k * L, l);
}
__device__ __forceinline__ BranchCoef branch_coef(const double2* br, int L, uint32_t l) {
    return {branch_pair(br, L, 0, l), branch_pair(br, L, 1, l), branch_pair(br, L, 2, l), branch_pair(br, L, 3, l)};
}

// The four flows of a branch at end voltages u, w and angle difference (C, S).
struct BranchFlows {
    PFlow pf, qf, pt, qt;
};
__device__ __forceinline__ BranchFlows branch_flows(const BranchCoef& k, double u, double w, double C, double S) {
    BranchFlows r;
    r.pf = pflow(k.ff.x, 0.0, k.ft.x, k.ft.y, u, w, C, S);
    r.qf = pflow(-k.ff.y, 0.0, -k.ft.y, k.ft.x, u, w, C, S);
    r.pt = pflow(0.0, k.tt.x, k.tf.x, -k.tf.y, u, w, C, S);
    r.qt = pflow(0.0, -k.tt.y, -k.tf.y, -k.tf.x, u, w, C, S);
    return r;
}

// What the gradient pass needs of a branch, kept in registers from the first
// pass: its end voltages, cos and sin of its angle difference, d loss / d its arc values (p_f,
// p_t, q_f, q_t) without the balance rows, the angle row's weight, and its end
// buses and half-edge positions.
struct BranchKeep {
    double u, w, C, S, ap[4], wa;
    int4 id;
};

// LDS, in pairs read and written by 16 bytes: (va, vm) [N]; (pg, qg) [G] in
// the bus-ordered generator list's order; (p, q) of each half-edge [2L] in the
// bus-ordered half-edge list's order (later the half-edge gradient terms
// d/dva, d/dvm), so that a bus sums one contiguous range; the balance rows'
// weights [N]; then the squashing activations [2N + 2G] (z's order) and the
// partial sums.  Sums run in the adjacency and generator-list orders;
// the loss in LANES lanes (a multiple of NT: a thread holds the lanes
// LANES / NT apart; buses and generators counted from the last lane), then
// over the lanes of each 64 in a fixed order, then over those in order.  So a
// sample's loss is the same bits in every launch shape of its network's size.
//
// Bound by its FP64 and address instructions (half of a SIMD's time), then by
// the latency of each phase.  A thread owns KR branches (L <= NT * KR) and
// carries what the gradient pass needs of them in registers over the
// barriers; each branch's parameters are packed for 16-byte loads, with only
// the bounds that a static model can have (fill_bounds: arcs within +-rate,
// thermal rows in (-inf, 0], balance rows 0).
// Buses go to the threads from the last one down: the last waves have the
// fewest branches.  4096 samples of 300 buses and 406 branches: 82.3 us with
// the branch parameters in separate arrays, read in three passes; 57 with
// them packed and kept; 53.1 with pairs in LDS; 51.4 with the buses turned
// (its instructions alone take 32).  Loading ahead of the barriers (102
// registers) 57.2; one branch per thread in workgroups of 448 73.0.  64
// samples: 13.1 -> 7.7 us.
template <int NT, int KR, int LANES>
__global__ void __launch_bounds__(NT) loss_fused_kernel(DevModel m, ProxBox box, ProxRows rows, ProxPerm pm,
                                                        const float* __restrict__ z, const double* __restrict__ loads,
                                                        double rho, double obj_scale, double* __restrict__ loss,
                                                        double* __restrict__ cvio, double* __restrict__ gz,
                                                        double* __restrict__ X, double* __restrict__ C,
                                                        float* __restrict__ dz, double w) {
#pragma clang fp contract(off)
    extern __shared__ double2 lds2[];
    const int N = m.N, L = m.L, G = m.G, D = 2 * N + 2 * G;
    double2* s_v = lds2;
    double2* s_g = s_v + N;
    double2* s_h = s_g + G;
    double2* s_wb = s_h + 2 * L;
    double* s_act = reinterpret_cast<double*>(s_wb + N);
    double* s_red = s_act + D;
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    const float* zb = z + b * D;
    double* xb = X ? X + b * rows.n : nullptr;
    double* cb = C ? C + b * rows.m : nullptr;
    const double* pdb = loads + b * 2 * N;
    constexpr int U = LANES / NT;
    static_assert(U <= 2 && (KR == 1 || KR % U == 0), "branch r of a thread is in its lane r % U");
    double pen[U] = {}, fobj = 0.0, vio = 0.0;
    auto add = [&](int u, double v) {  // v into lane u of two: the other adds 0
        if constexpr (U == 1) {
            pen[0] += v;
        } else {
            pen[0] += u ? 0.0 : v;
            pen[1] += u ? v : 0.0;
        }
    };

    for (int e = tid; e < D; e += NT) {
        // entry e of (va, vm, pg, qg): the half of pair (e - first) or of the generator's position
        const int pair = e < 2 * N ? (e < N ? e : e - N)
                                   : N + at(pm.gen_pos, e < 2 * N + G ? e - 2 * N : e - 2 * N - G);
        const int half = e < 2 * N ? e >= N : e >= 2 * N + G;
        double act;
        const double v = squash_entry(box, zb, e, act);
        reinterpret_cast<double*>(s_v)[2 * pair + half] = v;
        s_act[e < N ? N + e : (e < 2 * N ? e - N : e)] = act;
        if (xb) xb[e] = v;
    }
    __syncthreads();

    // branches: arc flows, the angle and thermal rows, the arc bounds
    const bool grad = gz || dz;
    BranchKeep keep[KR];
#pragma unroll
    for (int r = 0; r < KR; r++) {
        const uint32_t l = tid + r * NT;
        if (l >= (uint32_t)L) break;
        BranchKeep& t = keep[r];
        t.id = at(reinterpret_cast<const int4*>(pm.br + (size_t)6 * L), l);
        const BranchCoef k = branch_coef(pm.br, L, l);
        const double2 ang = branch_pair(pm.br, L, 4, l), rate = branch_pair(pm.br, L, 5, l);
        const double2 vf = s_v[t.id.x], vt = s_v[t.id.y];
        const double ca = vf.x - vt.x;
        t.u = vf.y;
        t.w = vt.y;
        sincos(ca, &t.S, &t.C);
        const BranchFlows f = branch_flows(k, t.u, t.w, t.C, t.S);
        s_h[t.id.z] = {f.pf.F, f.qf.F};
        s_h[t.id.w] = {f.pt.F, f.qt.F};
        const double arc[4] = {f.pf.F, f.pt.F, f.qf.F, f.qt.F};  // x's order
        const double cf = arc[0] * arc[0] + arc[2] * arc[2] - rate.y;
        const double ct = arc[1] * arc[1] + arc[3] * arc[3] - rate.y;
        const double dvf = cf > 0.0 ? cf : 0.0, dvt = ct > 0.0 ? ct : 0.0, dva = viol(ca, ang.x, ang.y);
        pen[r % U] += dvf * dvf;
        pen[r % U] += dvt * dvt;
        pen[r % U] += dva * dva;
        vio = fmax(vio, fmax(dvf, fmax(dvt, fabs(dva))));
        t.wa = 2.0 * rho * dva;
        const double wth[2] = {2.0 * rho * dvf, 2.0 * rho * dvt};
#pragma unroll
        for (int a = 0; a < 4; a++) {
            const double dq = viol(arc[a], -rate.x, rate.x);
            pen[r % U] += dq * dq;
            vio = fmax(vio, fabs(dq));
            t.ap[a] = 2.0 * arc[a] * wth[a & 1] + 2.0 * rho * dq;
        }
        if (xb) {
#pragma unroll
            for (int a = 0; a < 4; a++) xb[rows.pq0 + a * L + l] = arc[a];
        }
        if (cb) {  // flow rows: p - F(v) with p := F(v), exactly 0
            cb[m.c_pfr + l] = 0.0;
            cb[m.c_qfr + l] = 0.0;
            cb[m.c_pto + l] = 0.0;
            cb[m.c_qto + l] = 0.0;
            cb[m.c_ang + l] = ca;
            cb[m.c_thf + l] = cf;
            cb[m.c_tht + l] = ct;
        }
    }
    // objective terms (of two lanes the last: G <= NT) and reference rows
    for (int k = NT - 1 - tid; k < G; k += NT) {
        const double pg = s_g[at(pm.gen_pos, k)].x;
        fobj += at(m.c2, k) * pg * pg + at(m.c1, k) * pg + at(m.c0, k);
    }
    for (int q = tid, u = 0; q < m.R; q += NT, u ^= U - 1) {
        const double c = s_v[m.ref_bus[q]].x;
        const double dv = viol(c, rows.lcon[m.c_ref + q], rows.ucon[m.c_ref + q]);
        add(u, dv * dv);
        vio = fmax(vio, fabs(dv));
        if (cb) cb[m.c_ref + q] = c;
    }
    __syncthreads();

    // buses: balance rows, summed over contiguous half-edge and generator ranges
    for (int i = NT - 1 - tid, u = U - 1; i < N; i += NT, u ^= U - 1) {
        const int h0 = at(m.adj_ptr, i), h1 = at(m.adj_ptr, i + 1), g0 = at(m.gen_ptr, i), g1 = at(m.gen_ptr, i + 1);
        const double gs = at(m.gs, i), bs = at(m.bs, i), pd = at(pdb, i), qd = at(pdb, N + i);
        const double vm = s_v[i].y, v2 = vm * vm;
        double sp = 0.0, sq = 0.0;
        for (int h = h0; h < h1; h++) {
            const double2 v = s_h[h];
            sp += v.x;
            sq += v.y;
        }
        double cp = pd + gs * v2 + sp, cq = qd - bs * v2 + sq;
        for (int q = g0; q < g1; q++) {
            const double2 v = s_g[q];
            cp -= v.x;
            cq -= v.y;
        }
        const double dvp = viol(cp, 0.0, 0.0), dvq = viol(cq, 0.0, 0.0);
        add(u, dvp * dvp);
        add(u, dvq * dvq);
        vio = fmax(vio, fmax(fabs(dvp), fabs(dvq)));
        s_wb[i] = {2.0 * rho * dvp, 2.0 * rho * dvq};
        if (cb) {
            cb[m.c_balp + i] = cp;
            cb[m.c_balq + i] = cq;
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
#pragma unroll
        for (int u = 0; u < U; u++) pen[u] += __shfl_down(pen[u], d, 64);
        fobj += __shfl_down(fobj, d, 64);
        vio = fmax(vio, __shfl_down(vio, d, 64));
    }
    if ((tid & 63) == 0) {
        const int wave = tid >> 6;
#pragma unroll
        for (int u = 0; u < U; u++) s_red[u * (NT / 64) + wave] = pen[u];
        s_red[LANES / 64 + wave] = fobj;
        s_red[(LANES + NT) / 64 + wave] = vio;
    }
    __syncthreads();  // also: every balance weight written, every half-edge value read
    if (tid == 0) {
        double P = 0.0, F = 0.0, V = 0.0;
        for (int w = 0; w < LANES / 64; w++) P += s_red[w];
        for (int w = 0; w < NT / 64; w++) {
            F += s_red[LANES / 64 + w];
            V = fmax(V, s_red[(LANES + NT) / 64 + w]);
        }
        loss[b] = rho * P + obj_scale * F;
        cvio[b] = V;
    }
    if (!grad) return;

    // branches: d loss / d arc with the balance rows, carried through p = F(v)
    // to the branch's four voltage entries, per half-edge
#pragma unroll
    for (int r = 0; r < KR; r++) {
        const uint32_t l = tid + r * NT;
        if (l >= (uint32_t)L) break;
        const BranchKeep& t = keep[r];
        const BranchFlows f = branch_flows(branch_coef(pm.br, L, l), t.u, t.w, t.C, t.S);
        const double2 wf = s_wb[t.id.x], wt = s_wb[t.id.y];
        const double tpf = t.ap[0] + wf.x, tpt = t.ap[1] + wt.x;
        const double tqf = t.ap[2] + wf.y, tqt = t.ap[3] + wt.y;
        const double gt = tpf * f.pf.Ft + tqf * f.qf.Ft + tpt * f.pt.Ft + tqt * f.qt.Ft;
        s_h[t.id.z] = {gt + t.wa, tpf * f.pf.Fu + tqf * f.qf.Fu + tpt * f.pt.Fu + tqt * f.qt.Fu};
        s_h[t.id.w] = {-(gt + t.wa), tpf * f.pf.Fw + tqf * f.qf.Fw + tpt * f.pt.Fw + tqt * f.qt.Fw};
    }
    __syncthreads();
    // d loss / d z in FP64, or (dz) as (float)(w * d loss / d z): the scaling
    // pass's value written here directly
    auto put = [&](int j, double v) {
        if (dz)
            dz[b * D + j] = (float)(w * v);
        else
            gz[b * D + j] = v;
    };
    for (int i = NT - 1 - tid; i < N; i += NT) {
        const int h0 = at(m.adj_ptr, i), h1 = at(m.adj_ptr, i + 1);
        const double gs = at(m.gs, i), bs = at(m.bs, i);
        const double span_v = at(box.vmax, i) - at(box.vmin, i);
        const int ref = at(box.is_ref, i);
        double ga = 0.0, gm = 0.0;
        for (int h = h0; h < h1; h++) {
            const double2 v = s_h[h];
            ga += v.x;
            gm += v.y;
        }
        const double vm = s_v[i].y;
        const double2 wb = s_wb[i];
        gm += 2.0 * gs * vm * wb.x - 2.0 * bs * vm * wb.y;
        const double s = s_act[i];
        put(i, gm * span_v * s * (1.0 - s));
        const double t = s_act[N + i];
        put(N + i, ref ? 0.0 : ga * box.va_span * (1.0 - t * t));
    }
    for (int k = tid; k < G; k += NT) {
        const int bus = at(m.gen_bus, k), q = at(pm.gen_pos, k);
        const double2 wb = s_wb[bus];
        const double gp = -wb.x + obj_scale * (2.0 * at(m.c2, k) * s_g[q].x + at(m.c1, k));
        const double gq = -wb.y;
        const double sp = s_act[2 * N + k], sq = s_act[2 * N + G + k];
        put(2 * N + k, gp * (at(box.pmax, k) - at(box.pmin, k)) * sp * (1.0 - sp));
        put(2 * N + G + k, gq * (at(box.qmax, k) - at(box.qmin, k)) * sq * (1.0 - sq));
    }
}

// dz [B, D] = (float)(w_b * gz[b, j]) with w_b = wb[b], or the constant w
// when wb is NULL
__global__ void scale_rows_kernel(const double* __restrict__ gz, const double* __restrict__ wb, double w, int B,
                                  int D, float* __restrict__ dz) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)B * D) return;
    dz[idx] = (float)((wb ? wb[idx / D] : w) * gz[idx]);
}

}  // namespace

hipError_t prox_vjp_sum(const double* X, const double* gX1, const double* gX2, const ProxObj& ob, double obj_scale,
                        const double* wb, int B, int64_t n, int64_t nfree, double* gX, hipStream_t s) {
    const int64_t tot = (int64_t)B * n;
    hipLaunchKernelGGL(vjp_sum_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, X, gX1, gX2, ob, obj_scale,
                       wb, B, n, nfree, gX);
    return hipGetLastError();
}

int prox_gemm_splits(int M, int N, int K) {
    // enough 128 x 128 tiles for one per compute unit, each part at least 4 k tiles
    const int64_t blocks = (int64_t)((M + BM - 1) / BM) * ((N + 127) / 128);
    int s = 1;
    while (blocks * s < 256 && K >= 2 * s * 4 * BK && s < 16) s *= 2;
    return s;
}

namespace {
template <int BN, typename TA, typename TB, typename TACT>
void launch_gemm(int variant, dim3 grid, hipStream_t s, const TA* A, int lda, const TB* B, int ldb, float* C, int ldc,
                 int M, int N, int K, int kchunk, const float* bias, TACT* act, int accumulate, float* part) {
    const dim3 block(GEMM_THREADS);
    switch (variant) {
    case 0: hipLaunchKernelGGL((gemm_kernel<true, true, BN, TA, TB, TACT>), grid, block, 0, s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, accumulate, part); break;
    case 1: hipLaunchKernelGGL((gemm_kernel<true, false, BN, TA, TB, TACT>), grid, block, 0, s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, accumulate, part); break;
    case 2: hipLaunchKernelGGL((gemm_kernel<false, false, BN, TA, TB, TACT>), grid, block, 0, s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, accumulate, part); break;
    default: hipLaunchKernelGGL((gemm_kernel<false, true, BN, TA, TB, TACT>), grid, block, 0, s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, accumulate, part); break;
    }
}

constexpr int kUnits = 256;
int64_t tile_count(int M, int N, int z, int bm, int bn) {
    return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * z;
}
// Whether 128 x 128 tiles, two workgroups per compute unit, come in whole
// rounds: the last one more than half full.
bool whole_rounds(int64_t wide) {
    return wide >= 2 * kUnits && (wide % (2 * kUnits) == 0 || wide % (2 * kUnits) > kUnits);
}
// Whether an FP32 A takes the tiled kernels (out: bytes stored per row and
// column beside C's 4, for the activation).  Its tiles (128 x 128 beyond a
// round) fit one workgroup per unit, and every wave column reads and rounds
// A's values again, so beyond one round they lose to the register-staged
// kernel (which rounds them once, two or three workgroups per unit) where
// its rounds are whole: forward 8192 x 1024 x 1024 30.6 us, 35.4 in tiles,
// 4096 x 4096 x 4096 180 and 196; up to 384 tiles (its 64-column tiles are one
// round) only for short k loops: 6000 x 1024 x 256 13.7 and 15.5, x 1024 30.5
// and 29.7; and where one k tile is all (4096 x 512 x 64 5.7 and 6.0).  Between
// its rounds the tiles win (12000 x 1024 x 1024 with GELU 61.9 and 56.8;
// 10000 x 600 x 1024 48.0 and 35.6), with an activation once A and the
// outputs pass the last-level cache (32768 x 1024 x 600 145 and 112, x 256
// 68 and 74), and in the dh product (B read by the transpose read) from 1024
// k values on (8192 x 2048 x 2048 112.8, 107.7).
bool tiled_fp32(int variant, int M, int N, int k, int splits, int out) {
    const int64_t wide = tile_count(M, N, splits, 128, 128);
    if (!out && k <= 64 && tile_count(M, N, splits, 64, 64) > kUnits) return false;
    if (wide <= kUnits) return true;
    if (whole_rounds(wide))
        return (variant == 1 && k >= 1024) || (out && (int64_t)M * (4 * (int64_t)k + (4 + out) * (int64_t)N) > (256 << 20));
    return wide > 3 * kUnits / 2 || k >= 1024;
}

// Whether a product's operands allow the tiled kernels: 16-byte copies of
// whole chunks at 16-byte addresses (a row-contiguous operand: rows and
// leading dimension multiples of 8; a k-contiguous one: k values likewise, 4
// for FP32), and 32-bit offsets inside a tile.  FP32 operands only as a
// k-contiguous A: the transpose read moves 16-bit values.
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool tiled_operand(const void* p, bool bf16, bool k_cont, int ld, int rows, int K) {
    if (!aligned16(p) || ld > (1 << 20)) return false;
    const int unit = bf16 ? 8 : 4;
    return ld % unit == 0 && (k_cont ? K % unit == 0 : bf16 && rows % 8 == 0);
}
bool tiled_operands(int variant, const void* A, bool a_bf16, int lda, const void* B, bool b_bf16, int ldb, int M, int N,
                    int K) {
    if (variant > 2 || !b_bf16 || (variant == 2 && !a_bf16)) return false;
    return tiled_operand(A, a_bf16, variant != 2, lda, M, K) && tiled_operand(B, b_bf16, variant == 0, ldb, N, K);
}
bool tiled_product(int variant, const void* A, bool a_bf16, int lda, const void* B, bool b_bf16, int ldb, int M, int N,
                   int K, int splits, int out) {
    return tiled_operands(variant, A, a_bf16, lda, B, b_bf16, ldb, M, N, K) &&
           (a_bf16 || tiled_fp32(variant, M, N, K / splits, splits, out));
}

// Tile shapes: the smallest that needs no more workgroups than the chip has
// compute units (256), else the widest.  A workgroup's time is its k loop,
// bound by the rate a compute unit fills its LDS (about 45 bytes a clock from
// L2, less from beyond), and a smaller tile spreads the operands over more of
// them; beyond one round a wide tile moves the fewest bytes per product.
// Forward with GELU, 1024 k: 64 rows x 1024 columns 14.7 us in the
// register-staged kernel, 6.2 (32 x 32 tiles), 6.7 (64 x 64); 1024 rows 8.7
// (64 x 64), 9.4 (32 x 32), 10.2 (128 x 64), before 19.9; 4096 rows 16.6
// (128 x 64, two workgroups per unit), 17.3 (128 x 128, one), 21.2 (64 x 64),
// before 25.0.  Where 128 x 128 tiles of two stages, four waves of 64 x 64 and
// two workgroups per unit come in whole rounds they read a quarter fewer bytes
// per product: 4096 x 4096 x 4096 195 -> 136 us (the register-staged kernel
// 164; 128 x 128 of three stages and eight waves 170), 8192 x 1024 x 1024 27.2 ->
// 23.7 (28.3).  Where the last half of the columns would be empty, in between, and under a GELU epilogue of a short k loop, the
// narrower tile's smaller steps win (16384 x 600 x 600 with GELU 32.3, 39.3).
template <typename TA, bool AK, bool BK, int TM, int TN, int WM, int WN, int ST>
void tile_launch(hipStream_t s, const TA* A, int lda, const __bf16* B, int ldb, float* C, int ldc, int M, int N, int K,
                 int kchunk, const float* bias, void* act, bool act_bf16, int accumulate, int splits, float* work) {
    hipLaunchKernelGGL((tile_gemm_kernel<TA, AK, __bf16, BK, TM, TN, WM, WN, ST>),
                       dim3((N + TN - 1) / TN, (M + TM - 1) / TM, splits), dim3(64 * WM * WN), 0, s, A, lda, B, ldb, C,
                       ldc, M, N, K, kchunk, bias, act, act_bf16 ? 1 : 0, accumulate, work);
}
template <typename TA, bool AK, bool BK>
void tile_shape(hipStream_t s, const TA* A, int lda, const __bf16* B, int ldb, float* C, int ldc, int M, int N, int K,
                int kchunk, const float* bias, void* act, bool act_bf16, int accumulate, int splits, float* work) {
    if (tile_count(M, N, splits, 32, 32) <= kUnits)
        tile_launch<TA, AK, BK, 32, 32, 1, 1, 4>(s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16,
                                                 accumulate, splits, work);
    else if (tile_count(M, N, splits, 64, 64) <= kUnits)
        tile_launch<TA, AK, BK, 64, 64, 2, 2, 4>(s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16,
                                                 accumulate, splits, work);
    else if constexpr (sizeof(TA) == 4)  // twice the bytes per stage: one workgroup of 144 KiB per unit; each
                                         // value of A read and rounded by two waves (by four: 5 to 12 % slower)
        tile_launch<TA, AK, BK, 128, 128, 4, 2, 3>(s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16,
                                                   accumulate, splits, work);
    else if (const int64_t wide = tile_count(M, N, splits, 128, 128);
             whole_rounds(wide) && (!act || K >= 1024) && 15 * wide <= 8 * tile_count(M, N, splits, 128, 64))
        tile_launch<TA, AK, BK, 128, 128, 2, 2, 2>(s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16,
                                                   accumulate, splits, work);
    else
        tile_launch<TA, AK, BK, 128, 64, 4, 2, 3>(s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16,
                                                  accumulate, splits, work);
}
void tile_product(int variant, const void* A, bool a_bf16, int lda, const void* B, int ldb, float* C, int ldc, int M,
                  int N, int K, int kchunk, const float* bias, void* act, bool act_bf16, int accumulate, int splits,
                  float* work, hipStream_t s) {
    const __bf16* b = static_cast<const __bf16*>(B);
    if (!a_bf16) {
        const float* a = static_cast<const float*>(A);
        if (variant == 0)
            tile_shape<float, true, true>(s, a, lda, b, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16, accumulate,
                                          splits, work);
        else
            tile_shape<float, true, false>(s, a, lda, b, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16, accumulate,
                                           splits, work);
        return;
    }
    const __bf16* a = static_cast<const __bf16*>(A);
    if (variant == 0)
        tile_shape<__bf16, true, true>(s, a, lda, b, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16, accumulate,
                                       splits, work);
    else if (variant == 1)
        tile_shape<__bf16, true, false>(s, a, lda, b, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16, accumulate,
                                        splits, work);
    else
        tile_shape<__bf16, false, false>(s, a, lda, b, ldb, C, ldc, M, N, K, kchunk, bias, act, act_bf16, accumulate,
                                         splits, work);
}

int split_chunk(int K, int splits) { return splits == 1 ? K : ((K + splits - 1) / splits + BK - 1) / BK * BK; }

template <typename TACT>
hipError_t splitk_sum(const float* work, int splits, int M, int N, float* C, int ldc, const float* bias, TACT* act,
                      int accumulate, hipStream_t s) {
    const int64_t tot = (int64_t)M * (N / 4);
    hipLaunchKernelGGL(splitk_sum_kernel<TACT>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, work, splits, M,
                       N, C, ldc, bias, act, accumulate);
    return hipGetLastError();
}

template <typename TA, typename TB, typename TACT>
hipError_t gemm_typed(int variant, const TA* A, int lda, const TB* B, int ldb, float* C, int ldc, int M, int N, int K,
                      const float* bias, TACT* act, int accumulate, int splits, float* work, hipStream_t s,
                      bool finish = true) {
    if (splits < 1) splits = 1;
    const int kchunk = split_chunk(K, splits);
    float* part = splits == 1 ? nullptr : work;
    const int my = (M + BM - 1) / BM;
    // 128-column tiles when they already give two workgroups per CU, else
    // 64-column tiles (twice the workgroups, two resident per CU)
    const int64_t wide = (int64_t)my * ((N + 127) / 128) * splits;
    if (wide >= kWideMin)
        launch_gemm<128>(variant, dim3((N + 127) / 128, my, splits), s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias,
                         act, accumulate, part);
    else
        launch_gemm<64>(variant, dim3((N + 63) / 64, my, splits), s, A, lda, B, ldb, C, ldc, M, N, K, kchunk, bias,
                        act, accumulate, part);
    if (splits > 1 && finish) return splitk_sum(work, splits, M, N, C, ldc, bias, act, accumulate, s);
    return hipGetLastError();
}

template <typename TA, typename TB>
hipError_t gemm_act(int variant, const TA* A, int lda, const TB* B, int ldb, float* C, int ldc, int M, int N, int K,
                    const float* bias, void* act, bool act_bf16, int accumulate, int splits, float* work,
                    hipStream_t s, bool finish = true) {
    if (act_bf16)
        return gemm_typed(variant, A, lda, B, ldb, C, ldc, M, N, K, bias, static_cast<__bf16*>(act), accumulate, splits,
                          work, s, finish);
    return gemm_typed(variant, A, lda, B, ldb, C, ldc, M, N, K, bias, static_cast<float*>(act), accumulate, splits,
                      work, s, finish);
}

template <typename TA>
hipError_t gemm_b(int variant, const TA* A, int lda, const void* B, bool b_bf16, int ldb, float* C, int ldc, int M,
                  int N, int K, const float* bias, void* act, bool act_bf16, int accumulate, int splits, float* work,
                  hipStream_t s, bool finish = true) {
    if (b_bf16)
        return gemm_act(variant, A, lda, static_cast<const __bf16*>(B), ldb, C, ldc, M, N, K, bias, act, act_bf16,
                        accumulate, splits, work, s, finish);
    return gemm_act(variant, A, lda, static_cast<const float*>(B), ldb, C, ldc, M, N, K, bias, act, act_bf16,
                    accumulate, splits, work, s, finish);
}
}  // namespace

namespace {
template <typename TA, typename TB>
hipError_t gelu_bwd_typed(const TA* A, int lda, const TB* B, int ldb, const float* pre, int ldp, __bf16* out, int ldo,
                          int M, int N, int K, float* part, hipStream_t s) {
    hipLaunchKernelGGL((gemm_gelu_bwd_kernel<true, false, TA, TB>), dim3((N + 63) / 64, (M + BM - 1) / BM, 1),
                       dim3(GEMM_THREADS), 0, s, A, lda, B, ldb, pre, ldp, out, ldo, M, N, K, part);
    return hipGetLastError();
}
template <typename TA>
hipError_t gelu_bwd_b(const TA* A, int lda, const void* B, bool b_bf16, int ldb, const float* pre, int ldp, __bf16* out,
                      int ldo, int M, int N, int K, float* part, hipStream_t s) {
    if (b_bf16)
        return gelu_bwd_typed(A, lda, static_cast<const __bf16*>(B), ldb, pre, ldp, out, ldo, M, N, K, part, s);
    return gelu_bwd_typed(A, lda, static_cast<const float*>(B), ldb, pre, ldp, out, ldo, M, N, K, part, s);
}
}  // namespace

hipError_t prox_gemm_gelu_bwd(const void* A, bool a_bf16, int lda, const void* B, bool b_bf16, int ldb,
                              const float* pre, int ldp, void* out, int ldo, int M, int N, int K, float* part,
                              hipStream_t s) {
    __bf16* o = static_cast<__bf16*>(out);
    // Column width by the tile_shape rule (the column sums fix 128 rows):
    // 4096 x 1024 x 1024 19.6 us with 64 columns, 21.0 with 128, before 29.4;
    // 1024 rows 10.7 with 32, 11.7 with 64, before 24.9.
    if (tiled_operands(1, A, a_bf16, lda, B, b_bf16, ldb, M, N, K)) {
        const __bf16* b = static_cast<const __bf16*>(B);
        auto go = [&](auto kernel, const auto* a, int cols, int threads) {
            hipLaunchKernelGGL(kernel, dim3((N + cols - 1) / cols, (M + BM - 1) / BM, 1), dim3(threads), 0, s, a, lda, b,
                               ldb, pre, ldp, o, ldo, M, N, K, part);
        };
        if (a_bf16) {
            const __bf16* a = static_cast<const __bf16*>(A);
            if (tile_count(M, N, 1, BM, 32) <= kUnits)
                go(tile_gelu_bwd_kernel<__bf16, __bf16, 32, 4, 1, 3>, a, 32, 256);
            else
                go(tile_gelu_bwd_kernel<__bf16, __bf16, 64, 4, 2, 3>, a, 64, 512);
        } else {
            const float* a = static_cast<const float*>(A);
            if (tile_count(M, N, 1, BM, 64) <= kUnits)
                go(tile_gelu_bwd_kernel<float, __bf16, 64, 4, 2, 3>, a, 64, 512);
            else
                go(tile_gelu_bwd_kernel<float, __bf16, 128, 2, 4, 3>, a, 128, 512);
        }
        return hipGetLastError();
    }
    if (a_bf16)
        return gelu_bwd_b(static_cast<const __bf16*>(A), lda, B, b_bf16, ldb, pre, ldp, o, ldo, M, N, K, part, s);
    return gelu_bwd_b(static_cast<const float*>(A), lda, B, b_bf16, ldb, pre, ldp, o, ldo, M, N, K, part, s);
}

hipError_t prox_colsum_parts(const float* part, int chunks, int N, float* out, float scale, hipStream_t s) {
    hipLaunchKernelGGL(colsum_final_kernel, dim3((N + 63) / 64), dim3(256), 0, s, part, chunks, N, out, scale);
    return hipGetLastError();
}

hipError_t prox_gemm_mixed(int variant, const void* A, bool a_bf16, int lda, const void* B, bool b_bf16, int ldb,
                           float* C, int ldc, int M, int N, int K, const float* bias, void* act, bool act_bf16,
                           int accumulate, int splits, float* work, hipStream_t s) {
    if (tiled_product(variant, A, a_bf16, lda, B, b_bf16, ldb, M, N, K, splits, act ? (act_bf16 ? 2 : 4) : 0)) {
        tile_product(variant, A, a_bf16, lda, B, ldb, C, ldc, M, N, K, split_chunk(K, splits), bias, act, act_bf16,
                     accumulate, splits, splits > 1 ? work : nullptr, s);
        if (splits > 1)
            return act_bf16 ? splitk_sum(work, splits, M, N, C, ldc, bias, static_cast<__bf16*>(act), accumulate, s)
                            : splitk_sum(work, splits, M, N, C, ldc, bias, static_cast<float*>(act), accumulate, s);
        return hipGetLastError();
    }
    if (a_bf16)
        return gemm_b(variant, static_cast<const __bf16*>(A), lda, B, b_bf16, ldb, C, ldc, M, N, K, bias, act, act_bf16,
                      accumulate, splits, work, s);
    return gemm_b(variant, static_cast<const float*>(A), lda, B, b_bf16, ldb, C, ldc, M, N, K, bias, act, act_bf16,
                  accumulate, splits, work, s);
}

hipError_t prox_gemm_split_parts(int variant, const void* A, bool a_bf16, int lda, const void* B, bool b_bf16, int ldb,
                                 int M, int N, int K, int splits, float* work, hipStream_t s) {
    if (tiled_product(variant, A, a_bf16, lda, B, b_bf16, ldb, M, N, K, splits, 0)) {
        tile_product(variant, A, a_bf16, lda, B, ldb, nullptr, N, M, N, K, split_chunk(K, splits), nullptr, nullptr,
                     false, 0, splits, work, s);
        return hipGetLastError();
    }
    if (a_bf16)
        return gemm_b(variant, static_cast<const __bf16*>(A), lda, B, b_bf16, ldb, nullptr, N, M, N, K, nullptr, nullptr,
                      false, 0, splits, work, s, false);
    return gemm_b(variant, static_cast<const float*>(A), lda, B, b_bf16, ldb, nullptr, N, M, N, K, nullptr, nullptr,
                  false, 0, splits, work, s, false);
}

hipError_t prox_update(UpdateLayers u, float* p, float* m1, float* m2, void* pb, float lr, float b1, float b2, float eps,
                       const int32_t* count, int32_t* step, hipStream_t s) {
    int blocks = 0;
    for (int k = 0; k < u.n; k++) {
        UpdateLayer& L = u.layer[k];
        L.first = blocks;
        L.weight_blocks = (int32_t)(((int64_t)L.fo * L.fi / 4 + 255) / 256);
        blocks += L.weight_blocks + (L.fo + 63) / 64;
    }
    const bool vec = aligned16(p) && aligned16(m1) && aligned16(m2);
    hipLaunchKernelGGL(vec ? update_kernel<true> : update_kernel<false>, dim3(blocks), dim3(256), 0, s, u, p, m1, m2,
                       static_cast<__bf16*>(pb), lr, b1, b2, eps, count, step);
    return hipGetLastError();
}

hipError_t prox_gemm(int variant, const float* A, int lda, const float* B, int ldb, float* C, int ldc, int M, int N,
                     int K, const float* bias, float* act, int accumulate, int splits, float* work, hipStream_t s) {
    return prox_gemm_mixed(variant, A, false, lda, B, false, ldb, C, ldc, M, N, K, bias, act, false, accumulate, splits,
                           work, s);
}

hipError_t prox_gelu_bwd(const float* pre, const float* dact, float* dpre, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gelu_bwd_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pre, dact, dpre, n);
    return hipGetLastError();
}

hipError_t prox_colsum_first(const float* X, int M, int N, float* part, void* Xb, const int32_t* step, int32_t* next,
                             hipStream_t s) {
    const int chunks = (M + COLSUM_ROWS - 1) / COLSUM_ROWS;
    hipLaunchKernelGGL(colsum_partial_kernel, dim3((N + 63) / 64, chunks), dim3(256), 0, s, X, M, N, part,
                       static_cast<__bf16*>(Xb), step, next);
    return hipGetLastError();
}

hipError_t prox_colsum(const float* X, int M, int N, float* part, float* out, float scale, hipStream_t s) {
    const int chunks = (M + COLSUM_ROWS - 1) / COLSUM_ROWS;
    hipLaunchKernelGGL(colsum_partial_kernel, dim3((N + 63) / 64, chunks), dim3(256), 0, s, X, M, N, part,
                       static_cast<__bf16*>(nullptr), static_cast<const int32_t*>(nullptr),
                       static_cast<int32_t*>(nullptr));
    hipLaunchKernelGGL(colsum_final_kernel, dim3((N + 63) / 64), dim3(256), 0, s, part, chunks, N, out, scale);
    return hipGetLastError();
}


hipError_t prox_adam(float* p, const float* g, float* m1, float* m2, int64_t n, float lr, float b1, float b2, float eps,
                     int step, void* pb, hipStream_t s) {
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, g, m1, m2, n, lr, b1, b2,
                       eps, c1, c2, static_cast<__bf16*>(pb));
    return hipGetLastError();
}

hipError_t prox_adam_dev(float* p, const float* g, float* m1, float* m2, int64_t n, float lr, float b1, float b2,
                         float eps, int32_t* step, void* pb, hipStream_t s) {
    auto a16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
    if (a16(p) && a16(g) && a16(m1) && a16(m2) && (reinterpret_cast<uintptr_t>(pb) & 7u) == 0) {
        const int64_t blocks = std::min<int64_t>((n / 4 + 255) / 256, 2048);
        hipLaunchKernelGGL(adam_dev4_kernel, dim3((unsigned)std::max<int64_t>(blocks, 1)), dim3(256), 0, s, p, g, m1,
                           m2, n, lr, b1, b2, eps, step, static_cast<__bf16*>(pb));
    } else {
        hipLaunchKernelGGL(adam_dev_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, g, m1, m2, n, lr,
                           b1, b2, eps, step, static_cast<__bf16*>(pb));
    }
    hipLaunchKernelGGL(step_bump_kernel, dim3(1), dim3(1), 0, s, step);
    return hipGetLastError();
}

hipError_t prox_to_bf16(const float* x, int64_t n, void* y, hipStream_t s) {
    // 16-byte loads and stores where the buffers allow them (2.4 M values: 5.2 us)
    if (n % 8 == 0 && aligned16(x) && aligned16(y)) {
        hipLaunchKernelGGL(to_bf16x8_kernel, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, s, x, n / 8,
                           static_cast<__bf16*>(y));
        return hipGetLastError();
    }
    hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, n, static_cast<__bf16*>(y));
    return hipGetLastError();
}

hipError_t prox_squash_fwd(const float* z, int B, const ProxBox& box, double* X, int64_t n, bool arcs, hipStream_t s) {
    const int64_t per = arcs ? n : 2 * (int64_t)box.N + 2 * box.G;
    const int64_t tot = (int64_t)B * per;
    hipLaunchKernelGGL(squash_fwd_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, z, B, box, X, n, per);
    return hipGetLastError();
}

hipError_t prox_squash_bwd(const float* z, int B, const ProxBox& box, const double* gX1, const double* gX2,
                           const double* gObj, double obj_scale, int64_t n, float* dz, float scale, hipStream_t s) {
    const int64_t tot = (int64_t)B * (2 * box.N + 2 * box.G);
    hipLaunchKernelGGL(squash_bwd_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, z, B, box, gX1, gX2,
                       gObj, obj_scale, n, dz, scale);
    return hipGetLastError();
}

hipError_t prox_loss_bwd(const float* z, int B, const ProxBox& box, const ProxObj& ob, const double* X,
                         const double* gX1, double obj_scale, const double* wb, int64_t n, float* dz, hipStream_t s) {
    const int64_t tot = (int64_t)B * (2 * box.N + 2 * box.G);
    hipLaunchKernelGGL(loss_bwd_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, z, B, box, ob, X, gX1,
                       obj_scale, wb, n, dz);
    return hipGetLastError();
}

hipError_t prox_penalty(const double* C, const double* X, const double* F, double obj_scale, const ProxRows& rows,
                        double rho, int B, double* pen, double* cvio, double* W, double* gpq, int vjp, hipStream_t s) {
    const size_t lds = gpq ? 0 : sizeof(double) * (size_t)rows.npq;
    // 1,024 threads per instance where each has a row of its own and two
    // instances per compute unit (32 waves) hold the whole batch, or where each
    // has four rows; else 512 where each of those has four.  100 buses (1,111 rows): 256 instances 5.6 us with
    // 256 threads, 5.1 us with 1,024; 1,024 instances 9.5 and 11.0 us; 4,096
    // 25.6, 30.1 with 512, 34.3 with 1,024.  14 buses (169 rows), 256
    // instances: 3.6 and 4.4 us.  300 buses (3,471 rows): 1,024 instances 22.2,
    // 21.2, 21.2 us with 256, 512 and 1,024; 4,096 114, 108, 111.  500 buses
    // (5,551 rows), 4,096 instances: 188, 176, 170.  1,000 buses: 256 instances
    // 33.5 and 18.6 us with 256 and 1,024, 1,024 instances 86.5 (90.2 with 512)
    // and 86.8.
    // The lanes of the sum follow the rows alone (four a thread cost 0.3 us at
    // 100 buses and 513 instances).
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(B), dim3(threads), lds, s, C, X, F, obj_scale, rows, rho, pen, cvio, W, gpq, vjp);
    };
    if (rows.m < 1024)
        go(penalty_kernel<256, 256>, 256);
    else if (B <= 2 * kUnits || rows.m >= 4096)
        go(penalty_kernel<1024, 1024>, 1024);
    else if (rows.m >= 2048)
        go(penalty_kernel<512, 1024>, 512);
    else
        go(penalty_kernel<256, 1024>, 256);
    return hipGetLastError();
}

hipError_t prox_vjp_weights(const double* X, const double* W, const double* gpq, const ProxRows& rows, int B,
                            double* Wt, hipStream_t s) {
    if (Wt != W) {
        const int64_t tot = (int64_t)B * rows.m;
        hipLaunchKernelGGL(copy_off_flow_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, W, rows, B, Wt);
    }
    const int64_t nfl = (int64_t)B * (rows.flow1 - rows.flow0);
    if (nfl > 0)
        hipLaunchKernelGGL(vjp_weights_kernel, dim3((unsigned)((nfl + 255) / 256)), dim3(256), 0, s, X, W, gpq, rows,
                           B, Wt);
    return hipGetLastError();
}


namespace {
template <int NT, int KR, int LANES>
void launch_loss_fused(const DevModel& m, const ProxBox& box, const ProxRows& rows, const ProxPerm& pm, const float* z,
                       const double* loads, int B, double rho, double obj_scale, double* loss, double* cvio, double* gz,
                       double* X, double* C, hipStream_t s, float* dz, double w) {
    const size_t lds = sizeof(double) * ((size_t)6 * m.N + 4 * (size_t)m.G + 4 * (size_t)m.L + (LANES + 2 * NT) / 64);
    hipLaunchKernelGGL((loss_fused_kernel<NT, KR, LANES>), dim3(B), dim3(NT), lds, s, m, box, rows, pm, z, loads, rho,
                       obj_scale, loss, cvio, gz, X, C, dz, w);
}
}  // namespace

bool prox_loss_fused_size(int N, int L, int G) {
    return sizeof(double) * ((size_t)6 * N + 4 * (size_t)G + 6 * (size_t)L + 12) <= kFusedLdsMax;  // so L < 1366
}

hipError_t prox_loss_fused(const DevModel& m, const ProxBox& box, const ProxRows& rows, const ProxPerm& pm,
                           const float* z, const double* loads, int B, double rho, double obj_scale, double* loss,
                           double* cvio, double* gz, double* X, double* C, hipStream_t s, float* dz, double w) {
    // Two branches per thread keep the most workgroups on a compute unit; up
    // to two samples per unit one branch per thread ends sooner (300 buses, 406
    // branches: 64 samples 7.7 us, 9.3 with two; 512 11.2 and 12.1; 1024 17.4
    // and 17.6; 4096 54.6 and 51.0).  Beyond 512 branches both are even while
    // the batch is small and two win after (541 branches, 4096 samples: 81.7,
    // 120 with one).  Up to 64 branches, one wave per sample once a unit has
    // more than four (14 buses, 4096 samples: 12.4 us against 19.6 with 256
    // threads; 1024: 7.8 and 8.1; 64: 7.3 and 6.7).
    // The lanes of the loss follow the network alone (the second lane of a
    // thread costs 0.7 us of 51 at 4096 samples of 300 buses); one wave's 128
    // are the first and the last 64 of 256, the others being empty at its
    // sizes, and two lanes keep the objective's sum in the last.
    const bool one_wave = m.L <= 64 && m.N <= 64 && m.G <= 64;
    auto* launch = one_wave && B > 4 * kUnits      ? launch_loss_fused<64, 1, 128>
                   : m.L <= 256                   ? launch_loss_fused<256, 1, 256>
                   : m.L <= 512 && (B <= 2 * kUnits || m.G > 256) ? launch_loss_fused<512, 1, 512>
                   : m.L <= 512                   ? launch_loss_fused<256, 2, 512>
                   : m.L <= 1024                  ? launch_loss_fused<512, 2, 512>
                                                  : launch_loss_fused<1024, 2, 1024>;
    launch(m, box, rows, pm, z, loads, B, rho, obj_scale, loss, cvio, gz, X, C, s, dz, w);
    return hipGetLastError();
}

hipError_t prox_sample_loads(const double* r, const double* base, const double* inv_scale, double spread, int B,
                             int N, double* loads, float* feats, hipStream_t s) {
    const int64_t tot = (int64_t)B * 2 * N;
    hipLaunchKernelGGL(sample_loads_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, r, base, inv_scale,
                       spread, B, N, loads, feats);
    return hipGetLastError();
}

hipError_t prox_scale_rows(const double* gz, const double* wb, double w, int B, int D, float* dz, hipStream_t s) {
    const int64_t tot = (int64_t)B * D;
    hipLaunchKernelGGL(scale_rows_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, gz, wb, w, B, D, dz);
    return hipGetLastError();
}

}  // namespace opf
