// Matrix-core product tiles fed by direct-to-LDS loads, for operands stored
// as BF16 (device code only; proxy_kernels.hip launches it).
//
// The k loop keeps several tiles of 64 k values in flight: each wave
// copies its share of a tile from global memory straight into LDS
// (global_load_lds, 16 bytes per lane, no registers), one barrier per tile,
// and the wait before it counts only the tile about to be read.  An operand
// that is contiguous along its rows (dy, W of dy W) is copied as it lies and
// transposed when it is read, by the LDS transpose read (ds_read_b64_tr_b16).
//
// What bounds it (clocks inside the kernel, taken at 4096 x 1024 x 1024 on
// BF16 tiles of 128 x 128, 8 waves and three stages, which that product took
// before 128 x 64): a tile of 64 k values takes about 820 clocks, 640 of
// them needed by the LDS reads and the products alone, 600 by the copies
// alone; before, with one tile in flight through registers, about 2,000.  The
// copies spread between the products because in one burst they queue up and
// hold the products back (1,100 clocks a tile).  Direct copies rather than
// registers leave the vector unit to the products (four fewer instructions
// per 16 bytes) and their latency to the counted waits.
//
// Every product is v_mfma_f32_32x32x16_bf16 with k ascending, one
// accumulator per output element: the same additions in the same order for
// every tile shape here and in the register-staged kernel, so all of them
// give the same bits.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace opf {
namespace tile {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;

constexpr int kDepth = 64;  // k values per LDS tile

// One operand's tile of ROWS rows (i of A, j of B) by kDepth k values in LDS,
// copied by the wave in pieces of 1 KiB (16 bytes per lane).
//  BF16, KCONT: rows of 64 k values; the 16-byte chunk c of row r sits at
//         c ^ ((r >> 1) & 7) (reads of 32 rows then spread over the banks).
//  BF16, else:  rows of ROWS values, one per k; chunks XORed by k so that the
//         four k rows of a transpose read fall on distinct banks.
//  FP32, KCONT: rows of 64 k values, chunk c of row r at c ^ (r & 15); the
//         values are rounded to BF16 (nearest even) when they are read.
template <typename T, bool KCONT, int ROWS>
struct Operand {
    static_assert(KCONT || sizeof(T) == 2, "an FP32 operand is k-contiguous");
    static constexpr int kBytes = ROWS * kDepth * (int)sizeof(T);
    static constexpr int kCopies = kBytes / 1024;

    __device__ static __forceinline__ int swz(int k) {
        return ROWS >= 128 ? (k & 3) << 2 : (ROWS == 64 ? ((k >> 1) & 1) << 2 : 0);
    }
    // Global element this lane copies in wave copy t: (row, k) inside the
    // tile (KCONT: consecutive k values from k; else: 8 rows from row).
    __device__ static __forceinline__ void source(int t, int lane, int& row, int& k) {
        if (sizeof(T) == 4) {
            row = t * 4 + lane / 16;
            k = ((lane % 16) ^ (row & 15)) * 4;
        } else if (KCONT) {
            row = t * 8 + lane / 8;
            k = ((lane % 8) ^ ((row >> 1) & 7)) * 8;
        } else {
            constexpr int CH = ROWS / 8;  // chunks per k row
            k = t * (64 / CH) + lane / CH;
            row = ((lane % CH) ^ swz(k)) * 8;
        }
    }
    // The MFMA operand of rows r0 .. r0 + 31 at k step ks (16 values).
    __device__ static __forceinline__ bf16x8 frag(const char* S, int r0, int ks, int lane) {
        if constexpr (sizeof(T) == 4) {
            const int r = r0 + lane % 32, c = (ks * 2 + lane / 32) * 2;
            const float4 u = *reinterpret_cast<const float4*>(S + r * 256 + ((c ^ (r & 15)) << 4));
            const float4 v = *reinterpret_cast<const float4*>(S + r * 256 + (((c + 1) ^ (r & 15)) << 4));
            return (bf16x8){(__bf16)u.x, (__bf16)u.y, (__bf16)u.z, (__bf16)u.w,
                            (__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
        } else if constexpr (KCONT) {
            const int r = r0 + lane % 32, c = ks * 2 + lane / 32;
            return *reinterpret_cast<const bf16x8*>(S + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
        } else {
            const int k = ks * 16 + 8 * (lane / 32) + (lane % 16) / 4;
            const int col = r0 + 16 * ((lane / 16) % 2) + 4 * (lane % 4);
            const char* p = S + k * (2 * ROWS) + (((col / 8) ^ swz(k)) << 4) + 2 * (col % 8);
            typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
            union {
                s16x4 h[2];
                bf16x8 v;
            } u;
            u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
            u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 8 * ROWS));
            return u.v;
        }
    }
};

__device__ __align__(16) static const uint4 kZeroChunk = {0u, 0u, 0u, 0u};

// 64 lanes x 16 bytes from each lane's p to LDS at the wave's base + 16 lane.
__device__ __forceinline__ void copy_lds(const void* p, char* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                     (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// s_waitcnt with vmcnt(N) and lgkmcnt(0); the other counters untouched.
template <int N>
__device__ __forceinline__ void wait_copies() {
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

// Workgroup barrier without the waits of __syncthreads (the copies in flight
// are waited for by count); no memory access moves across it.
__device__ __forceinline__ void barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// One wave's share of the copies of an operand: NI wave copies per tile.  The
// tile's origin is a uniform pointer, each lane's place in the tile a 32-bit
// byte offset that holds for every tile.
template <typename T, bool KCONT, int ROWS, int WAVES>
struct Copier {
    typedef Operand<T, KCONT, ROWS> Op;
    static constexpr int NI = Op::kCopies / WAVES;
    static_assert(NI * WAVES == Op::kCopies, "tile rows and waves");
    const char* base;  // the next tile's origin
    uint32_t off[NI];
    // rows past nrows read the last valid ones again: their products are never stored
    __device__ __forceinline__ void init(const T* P, int ld, int nrows, int r0, int kb, int wave, int lane) {
        base = reinterpret_cast<const char*>(KCONT ? P + (size_t)r0 * ld + kb : P + (size_t)kb * ld + r0);
#pragma unroll
        for (int q = 0; q < NI; q++) {
            int row, k;
            Op::source(wave * NI + q, lane, row, k);
            off[q] = (uint32_t)(KCONT ? min(row, nrows - 1 - r0) * ld + k : k * ld + min(row, nrows - 8 - r0)) *
                     (uint32_t)sizeof(T);
        }
    }
    __device__ __forceinline__ void advance(int ld) { base += (KCONT ? (size_t)kDepth : (size_t)kDepth * ld) * sizeof(T); }
    __device__ __forceinline__ void copy(char* S, int q, int wave) {
        copy_lds(base + off[q], S + (wave * NI + q) * 1024);
    }
    // the same where only `left` k values of the tile remain: zeros past them
    __device__ __forceinline__ void copy_part(char* S, int q, int left, int wave, int lane) {
        int row, k;
        Op::source(wave * NI + q, lane, row, k);
        const char* s = k < left ? base + off[q] : reinterpret_cast<const char*>(&kZeroChunk);
        copy_lds(s, S + (wave * NI + q) * 1024);
    }
};

// The kernel's only __shared__ array must be the one that holds the tiles: with
// several, the compiler waits for every copy in flight before each LDS read.
//
// The k loop of a BM x BN tile at (i0, j0) over k in [kb, ke): WM x WN waves
// of (BM / WM) x (BN / WN), accumulators acc[a][b] of 32 x 32.  Every wave of
// the workgroup is past its last LDS read on return.
template <typename TA, bool AK, typename TB, bool BK, int BM, int BN, int WM, int WN, int ST>
struct Tile {
    static constexpr int WAVES = WM * WN, NA = BM / WM / 32, NB = BN / WN / 32;
    typedef Copier<TA, AK, BM, WAVES> CA;
    typedef Copier<TB, BK, BN, WAVES> CB;
    static constexpr int kAt = CA::Op::kBytes;             // B's tile after A's
    static constexpr int kStage = kAt + CB::Op::kBytes;    // bytes of a stage
    static constexpr int kBytes = ST * kStage;
    static constexpr int kPer = CA::NI + CB::NI;  // copies per wave and tile
    static_assert(kPer * (ST - 1) < 64, "vmcnt range");

    // Waits until at most `later` tiles' copies of this wave are outstanding.
    template <int K>
    __device__ static __forceinline__ void wait_tiles(int later) {
        if constexpr (K == 0) {
            wait_copies<0>();
        } else if (later >= K) {
            wait_copies<K * kPer>();
        } else {
            wait_tiles<K - 1>(later);
        }
    }

    __device__ static __forceinline__ void run(const TA* __restrict__ A, int lda, const TB* __restrict__ B, int ldb,
                                               int M, int N, int i0, int j0, int kb, int ke, char* smem,
                                               f32x16 (&acc)[NA][NB]) {
        const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
        const int wi = (wave / WN) * (BM / WM), wj = (wave % WN) * (BN / WN);
#pragma unroll
        for (int a = 0; a < NA; a++)
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int v = 0; v < 16; v++) acc[a][b][v] = 0.f;
        CA ca;
        CB cb;
        ca.init(A, lda, M, i0, kb, wave, lane);
        cb.init(B, ldb, N, j0, kb, wave, lane);
        const int nt = (ke - kb + kDepth - 1) / kDepth;
        const int full = (ke - kb) / kDepth;  // tiles of kDepth values; a part tile may follow
        // copy c of this wave's kPer copies of the next whole tile
        auto copy = [&](int c, int buf) {
            char* S = smem + buf * kStage;
            if (c < CA::NI)
                ca.copy(S, c, wave);
            else
                cb.copy(S + kAt, c - CA::NI, wave);
        };
        // tile t (the next one) in one go
        auto issue = [&](int t, int buf) {
            if (t < full) {
#pragma unroll
                for (int c = 0; c < kPer; c++) copy(c, buf);
                ca.advance(lda);
                cb.advance(ldb);
            } else {
                char* S = smem + buf * kStage;
#pragma unroll
                for (int q = 0; q < CA::NI; q++) ca.copy_part(S, q, ke - kb - t * kDepth, wave, lane);
#pragma unroll
                for (int q = 0; q < CB::NI; q++) cb.copy_part(S + kAt, q, ke - kb - t * kDepth, wave, lane);
            }
        };
        // fragments of the four k steps of a tile, read two steps ahead of their products
        bf16x8 fa[4][NA], fb[4][NB];
        auto read = [&](int buf, int ks) {
            const char* SA = smem + buf * kStage;
            const char* SB = SA + kAt;
#pragma unroll
            for (int a = 0; a < NA; a++) fa[ks][a] = CA::Op::frag(SA, wi + a * 32, ks, lane);
#pragma unroll
            for (int b = 0; b < NB; b++) fb[ks][b] = CB::Op::frag(SB, wj + b * 32, ks, lane);
        };
        // the products of step ks; half >= 0: half of the next tile's copies between them
        constexpr int kMul = NA * NB;
        auto mul = [&](int ks, int half, int b0) {
#pragma unroll
            for (int a = 0; a < NA; a++)
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][a], fb[ks][b], acc[a][b], 0, 0, 0);
                    if (half >= 0) {
#pragma unroll
                        for (int c = 0; c < kPer; c++)
                            if (c * 2 * kMul / kPer == half * kMul + a * NB + b) copy(c, b0);
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        };
        if (nt == 0) return;
#pragma unroll
        for (int t = 0; t < ST; t++)
            if (t < nt) issue(t, t);
        wait_tiles<ST - 1>(nt - 1);
        barrier();
        read(0, 0);
        read(0, 1);
        // Tile t + ST goes where tile t was, its copies spread between the
        // products after the barrier that frees it (in one burst they would
        // hold the products back while they queue up).
        int buf = 0, t = 0;
        for (; t < full - ST; t++) {
            const int next = buf + 1 == ST ? 0 : buf + 1;
            read(buf, 2);
            mul(0, -1, 0);
            read(buf, 3);
            mul(1, -1, 0);
            // this wave's reads of tile t are done and its copies of tile t + 1 landed; after the
            // barrier every wave's are
            wait_copies<(ST - 2) * kPer>();
            barrier();
            read(next, 0);
            mul(2, 0, buf);
            read(next, 1);
            mul(3, 1, buf);
            ca.advance(lda);
            cb.advance(ldb);
            buf = next;
        }
        // the last ST tiles: nothing but a part tile left to copy
        for (; t < nt - 1; t++) {
            const int next = buf + 1 == ST ? 0 : buf + 1;
            read(buf, 2);
            mul(0, -1, 0);
            read(buf, 3);
            mul(1, -1, 0);
            wait_tiles<ST - 2>(min(nt - 2 - t, ST - 2));
            barrier();
            if (t + ST < nt) issue(t + ST, buf);
            read(next, 0);
            mul(2, -1, 0);
            read(next, 1);
            mul(3, -1, 0);
            buf = next;
        }
        read(buf, 2);
        mul(0, -1, 0);
        read(buf, 3);
        mul(1, -1, 0);
        mul(2, -1, 0);
        mul(3, -1, 0);
        wait_copies<0>();
        barrier();
    }
};

}  // namespace tile
}  // namespace opf
