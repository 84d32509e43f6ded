// ksplit_gemm.hpp - 16 x 16 tiles whose workgroup splits K over its waves.
//
// For products of few tiles and long K (decoding a few tokens against a
// narrow layer) the time is one wave's walk along K: a slice costs it an LDS
// read and two MFMAs in sequence, about 0.1 us, however few bytes that is.
// Here KS waves share one 16 x 16 tile, each walking its own contiguous part
// of the K-slices through its own eight-slice LDS ring (32 KiB), and add up
// at the end, in wave order, so results do not depend on timing. No wave
// touches another's ring, so the walk has no barrier at all: a wave waits for
// its own copies (vmcnt) and its own reads (lgkmcnt).
//
// Per slice: the reads of this slice (issued a slice ago) are in registers,
// so its buffer takes the copy of the slice eight further on; the next
// slice's copy has landed, its reads are issued; this slice's MFMAs run.
// The terms of scaled outputs are loaded before the walk.
//
// Graph replays on MI355X, us with one, two and four waves: INT4 32 x 4096 x
// 14336 (512 tiles) 13.3, 9.3, 12.0, FP16 4 x 2048 x 4096 (128 tiles) 9.0,
// 6.2, 5.5, INT4 16 x 4096 x 14336 12.9, 8.8, 8.3; no gain where memory is
// what takes the time (FP16 16 x 8192 x 8192 29.4, 30.6, 32.5) or the tiles
// fill the CUs by themselves (512^3 4.5, 5.7, 7.5).
#pragma once

#include "tiled_gemm.hpp"

namespace mpg {

typedef TileCfg<16, 16, 1, 1, 128, 8, 4, 16> KsCfg;

// Wait until the copies of at most `slices` later slices are in flight.
template <int MAX>
__device__ __forceinline__ void ks_wait(int slices) {
    if constexpr (MAX > 0) {
        if (slices >= MAX) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAX * KsCfg::DMA_PER_WAVE) : "memory");
            return;
        }
        ks_wait<MAX - 1>(slices);
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
}

// Slice kt of n: its runs are in (ca, cb), the next one's go to (na, nb).
template <int DT, bool ISSUE>
__device__ __forceinline__ void ks_slice(uint8_t *ring, const uint8_t *const *src, int kt, int n, int r, int h,
                                         const i32x4 (&ca)[2][1], const i32x4 (&cb)[2][1], i32x4 (&na)[2][1],
                                         i32x4 (&nb)[2][1], typename Acc<DT, 16>::type (&acc)[1][1]) {
    typedef KsCfg T;
    constexpr int S = T::STAGES;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this slice's runs have arrived
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (ISSUE) {
        issue_stage<T>(ring, src, 0, kt % S, kt + S);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * T::DMA_PER_WAVE) : "memory");
    } else {
        ks_wait<S - 1>(n - 2 - kt);
    }
    // (after the last slice this reads a buffer nobody uses again; harmless)
    const uint8_t *st = ring + ((kt + 1) % S) * T::STAGE_BYTES;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) load_runs<T>(st, kc, 0, 0, r, h, na[kc], nb[kc]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) mma_runs<DT, T, 0, 1>(ca[kc], cb[kc], acc);
}

template <int DT, int KS>
__global__ __launch_bounds__(64 * KS) void ksplit_gemm(const uint8_t *__restrict__ A, const uint8_t *__restrict__ B,
                                                       void *__restrict__ Cv, int M, int N, int Kb, int tiles_m,
                                                       int tiles_n, EpiParams epi) {
    typedef KsCfg T;
    typedef typename Acc<DT, 16>::type acc_t;
    typedef typename Acc<DT, 16>::out out_t;
    constexpr int S = T::STAGES, E = 256 / (64 * KS);  // elements of C per thread
    __shared__ __attribute__((aligned(1024))) uint8_t lds[KS * T::LDS_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, h = lane >> 4;
    int tm, tn;
    tile_coords(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, T::GROUP_M, tm, tn);

    const int KT = Kb / T::BKB;
    const int k0 = (int)((long)KT * wave / KS), n = (int)((long)KT * (wave + 1) / KS) - k0;
    uint8_t *ring = lds + wave * T::LDS_BYTES;
    const uint8_t *src[T::DMA_PER_WAVE];
#pragma unroll
    for (int j = 0; j < T::DMA_PER_WAVE; ++j)
        src[j] = stage_src<T>(A, B, M, N, Kb, tm, tn, j, lane) + (size_t)k0 * T::BKB;
    acc_t acc[1][1];
    acc[0][0] = acc_t{};
    const int primed = min(n, S);
    for (int s = 0; s < primed; ++s) issue_stage<T>(ring, src, 0, s, s);

    // element x of this thread: accumulator value v of lane l of the tile
    long row[E], col[E];
    EpiOne one[E];
#pragma unroll
    for (int x = 0; x < E; ++x) {
        const int e = tid + x * 64 * KS, l = e & 63;
        row[x] = (long)tm * 16 + acc_row<16>(l >> 4, e >> 6);
        col[x] = (long)tn * 16 + (l & 15);
        one[x] = epi_one_terms<DT>(epi, row[x], col[x], M, N);
    }

    if (n > 0) {
        ks_wait<S - 1>(n - 1);
        i32x4 a0[2][1], b0[2][1], a1[2][1], b1[2][1];
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) load_runs<T>(ring, kc, 0, 0, r, h, a0[kc], b0[kc]);
        int kt = 0;
        for (; kt + 1 + S < n; kt += 2) {
            ks_slice<DT, true>(ring, src, kt, n, r, h, a0, b0, a1, b1, acc);
            ks_slice<DT, true>(ring, src, kt + 1, n, r, h, a1, b1, a0, b0, acc);
        }
        // at most one more slice issues a copy; then the rest
        if (kt + S < n) ks_slice<DT, true>(ring, src, kt, n, r, h, a0, b0, a1, b1, acc);
        else ks_slice<DT, false>(ring, src, kt, n, r, h, a0, b0, a1, b1, acc);
        for (++kt; kt < n; kt += 2) {
            ks_slice<DT, false>(ring, src, kt, n, r, h, a1, b1, a0, b0, acc);
            if (kt + 1 >= n) break;
            ks_slice<DT, false>(ring, src, kt + 1, n, r, h, a0, b0, a1, b1, acc);
        }
    }

    // the waves' partial tiles through their own rings, added in wave order
    out_t *part = reinterpret_cast<out_t *>(ring);
#pragma unroll
    for (int v = 0; v < 4; ++v) part[v * 64 + lane] = (out_t)acc[0][0][v];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < E; ++x) {
        const int e = tid + x * 64 * KS;
        out_t s = reinterpret_cast<const out_t *>(lds)[e];
#pragma unroll
        for (int w = 1; w < KS; ++w) s += reinterpret_cast<const out_t *>(lds + w * T::LDS_BYTES)[e];
        if constexpr (DT == S4) s >>= 8;  // INT4 sums carried times 256
        if (row[x] < M && col[x] < N) epi_store_terms<DT>(epi, one[x], Cv, row[x], col[x], N, s);
    }
}

}  // namespace mpg
