// tposeb_gemm.hpp - B stored K x N row-major (N-contiguous): the paper's
// "transposed B" operand layout (its INT4 ablation, Table XII), on CDNA4.
//
// On the paper's GPU this layout made every B load uncoalesced and cost 3x.
// Here B is copied into LDS exactly as it lies in memory (whole K-rows of
// N-contiguous bytes, the same 16-byte direct-to-LDS loads as A), and the
// MFMA operand, which wants K-contiguous runs per column, is assembled by the
// LDS transpose reads of gfx950 (ds_read_b64_tr_b16 / _b8 / _b4). Measured
// lane layout of those reads, per group of 16 lanes: lanes 4e..4e+3 (b16),
// 2e, 2e+1 (b8) or e (b4) supply row e (16 consecutive elements, 8 bytes per
// lane); output lane i receives element i of every row, i.e. 4 (b16), 8 (b8)
// or 16 (b4, row e in nibble e) elements of column i along the row index.
// With the rows being consecutive k of one 16-column slice, each lane gets
// consecutive k of its own column: the MFMA operand run, two reads per
// 32-column block per K-chunk. For INT4 (B's nibbles packed along N, the
// low nibble holding the even column) the two reads give 32 consecutive k
// packed two per byte with the low nibble holding the even k, the layout of
// a column-major INT4 run, so the decode and MFMAs are the column-major
// kernel's.
//
// Everything else is the pipelined kernel of tiled_gemm.hpp: 128-byte
// K-slices of A (BKB / es k-rows of B), operand runs double-buffered in
// registers. Four tiles: 256 x 256 (8 waves of 128 x 64, two stages, runs read
// a K-chunk ahead, the barrier inside the last chunk) and, where those leave
// CUs idle, 128 x 128 (8 waves of 64 x 32), 64 x 128 and 64 x 64 (waves of 32
// x 32), four stages, runs read a whole slice ahead. What bounds the small
// ones is a workgroup's time per slice: 0.5-0.65 us with 128 x 128 tiles, 0.4
// with 64 x 64 (FP16; 0.85 and 0.58 read a chunk ahead), so 256 of them at
// once matter more than bytes: INT8 1024 x 4096 x 4096 56.5 -> 25.4 us, FP16
// 105 x 2560 x 4096 97.3 -> 26.0 against 256 x 256 tiles alone. FP16, INT8
// and INT4. N must fill whole tiles (the copy takes whole B rows), K whole
// slices; M may be ragged.
#pragma once

#include "tiled_gemm.hpp"

namespace mpg {

template <int DT, class T>
struct TB {
    static_assert(T::MS == 32 && T::BKB == 128, "32x32 MFMAs, 128-byte slices");
    static constexpr int EPB2 = DT == F16 ? 1 : (DT == S8 ? 2 : 4);  // elements per 2 bytes
    static constexpr int BK = T::BKB * EPB2 / 2;         // k per slice = B rows per stage
    static constexpr int RB = T::BN * 2 / EPB2;          // bytes of one B row in the tile
    static constexpr int CHB = RB / 16;                  // 16-byte chunks per B row
    static constexpr int ROWS_PER_UNIT = 1024 / RB;      // B rows one 1 KiB copy fills
    static constexpr int A_UNITS = T::BM * T::BKB / 1024;
    static constexpr int RR = 4 * EPB2;                  // B rows per transpose read: 4, 8, 16
    static constexpr int LPR = 16 / RR;                  // lanes per row in a 16-lane group
    // byte offset of column j within a B row
    static __host__ __device__ constexpr long col_bytes(long j) { return j * 2 / EPB2; }
    static_assert(BK * RB == T::BN * T::BKB, "B part of a stage is as large as the column-major one");
};

// Slot of 16-byte chunk c of B row r (row r of the stage's B part, RB bytes):
// c ^ tb_swz(r). Two neighbouring 16-lane groups of a transpose read take RR
// consecutive rows (4, 8, 16) of one 32-column slice: 64 (FP16), 32 (INT8) or
// 16 (INT4) bytes of each, 256 bytes in all. Rows start on the same bank
// every 256 / RB of them (every row from 256 bytes on), so the rows that
// share a start are spread over the chunks: the read touches all 64 banks once.
template <int DT, int RB>
__host__ __device__ constexpr int tb_swz(int r) {
    constexpr int SH = RB >= 256 ? 0 : (RB == 128 ? 1 : (RB == 64 ? 2 : 3)), CH = RB / 16 < 16 ? RB / 16 : 16;
    const int x = r >> SH;
    return (DT == F16 ? 4 * (x & 3) : (DT == S8 ? 2 * (x & 7) : (x & 15))) & (CH - 1);
}

// Copy unit d of a stage for lane `lane`: A units as in the pipelined kernel;
// B unit u (d = A_UNITS + u) takes B rows kt * BK + u * ROWS_PER_UNIT + ...,
// chunk slot lane % CHB holding logical chunk slot ^ tb_swz(row). Returns the
// source at slice 0 (tb_issue adds the per-slice advance).
template <int DT, class T>
__device__ __forceinline__ const uint8_t *tb_src(const uint8_t *A, const uint8_t *B, int M, int N,
                                                 int Kb, int tm, int tn, int d, int lane) {
    typedef TB<DT, T> P;
    if (d < P::A_UNITS) return stage_src<T>(A, B, M, N, Kb, tm, tn, d, lane);
    const int u = d - P::A_UNITS;
    const int r = u * P::ROWS_PER_UNIT + lane / P::CHB;  // B row within the stage
    const int c = (lane % P::CHB) ^ tb_swz<DT, P::RB>(r);
    return B + (size_t)r * P::col_bytes(N) + (size_t)tn * P::RB + c * 16;
}

// One K-chunk's operand runs: A by ds_read_b128 (as load_runs), B by two
// transpose reads per 32-column block.
template <int DT, class T>
__device__ __forceinline__ void tb_load_runs(const uint8_t *st, int kc, int wm, int wn, int lane,
                                             i32x4 (&a)[T::FM], i32x4 (&b)[T::FN]) {
    typedef TB<DT, T> P;
    const int r = lane % T::MS, h = lane / T::MS;
#pragma unroll
    for (int i = 0; i < T::FM; ++i) {
        const int q = wm * T::WTM + i * T::MS + r;
        a[i] = *reinterpret_cast<const i32x4 *>(st + q * T::BKB + (((T::G * kc + h) ^ swz<T::CH>(q)) << 4));
    }
    const uint8_t *sb = st + T::BM * T::BKB;  // B part of the stage
    const int g = lane >> 4, j16 = lane & 15;
#pragma unroll
    for (int j = 0; j < T::FN; ++j) {
        const int col = wn * T::WTN + j * T::MS + 16 * (g & 1);  // first column of the group
        const int byte = (int)P::col_bytes(col) + (j16 % P::LPR) * 8;  // this lane's 8 bytes in the row
        i32x4 v;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            // k rows of this read: chunk kc's 16 (FP16) / 32 (INT8) / 64 (INT4) k, half g / 2, part t
            const int row = kc * (2 * 2 * P::RR) + (g >> 1) * (2 * P::RR) + t * P::RR + j16 / P::LPR;
            const uint8_t *p = sb + row * P::RB + ((((byte >> 4) ^ tb_swz<DT, P::RB>(row))) << 4) + (byte & 15);
            typedef __attribute__((address_space(3))) void lds_void_t;
            if constexpr (DT == F16) {
                typedef short v4s __attribute__((ext_vector_type(4)));
                typedef __attribute__((address_space(3))) v4s lds_v4s;
                const v4s x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)(lds_void_t *)p);
                const uint64_t u = __builtin_bit_cast(uint64_t, x);
                v[2 * t] = (int)(uint32_t)u;
                v[2 * t + 1] = (int)(uint32_t)(u >> 32);
            } else if constexpr (DT == S8) {
                typedef int v2i __attribute__((ext_vector_type(2)));
                typedef __attribute__((address_space(3))) v2i lds_v2i;
                const v2i x = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(lds_void_t *)p);
                v[2 * t] = x[0];
                v[2 * t + 1] = x[1];
            } else {
                typedef int v2i __attribute__((ext_vector_type(2)));
                typedef __attribute__((address_space(3))) v2i lds_v2i;
                const v2i x = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i *)(lds_void_t *)p);
                v[2 * t] = x[0];
                v[2 * t + 1] = x[1];
            }
        }
        b[j] = v;
    }
}

// This wave's copies of slice kt into buffer `stage`: A units advance by the
// slice's bytes, B units by its BK rows (`stride` bytes).
template <int DT, class T>
__device__ __forceinline__ void tb_issue(uint8_t *lds, const uint8_t *const *src, int wave, int stage,
                                         int kt, long stride) {
#pragma unroll
    for (int j = 0; j < T::DMA_PER_WAVE; ++j) {
        const int d = wave * T::DMA_PER_WAVE + j;
        dma16(src[j] + kt * (d < TB<DT, T>::A_UNITS ? (long)T::BKB : stride), lds + stage * T::STAGE_BYTES + d * 1024);
    }
}

template <int DT, class T, bool ISSUE>
__device__ __forceinline__ void tb_slice(uint8_t *lds, const uint8_t *const *src, long stride, int wave,
                                         int kt, int wm, int wn, int lane, i32x4 (&ra)[2][T::FM],
                                         i32x4 (&rb)[2][T::FN], typename Acc<DT, 32>::type (&acc)[T::FM][T::FN]) {
    constexpr int NB = T::FM * T::FN;
    constexpr int NRD = T::FM + 2 * T::FN;  // LDS reads per K-chunk
    constexpr int S = T::STAGES;
    const uint8_t *st = lds + (kt % S) * T::STAGE_BYTES;
#pragma unroll
    for (int kc = 0; kc < T::KCH - 1; ++kc) {
        const int cur = kc & 1;
        __builtin_amdgcn_sched_barrier(0);
        tb_load_runs<DT, T>(st, kc + 1, wm, wn, lane, ra[cur ^ 1], rb[cur ^ 1]);
        mma_runs<DT, T, 0, NB>(ra[cur], rb[cur], acc);
        chunk_hint<NB, NRD < NB ? NRD : NB, 0>();
        __builtin_amdgcn_sched_barrier(0);
    }
    constexpr int last = (T::KCH - 1) & 1;
    constexpr int PRE = NB / 4;
    mma_runs<DT, T, 0, PRE>(ra[last], rb[last], acc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (ISSUE) wait_vm_barrier<(S - 2) * T::DMA_PER_WAVE>();
    else wait_vm_barrier<0>();
    if constexpr (ISSUE) tb_issue<DT, T>(lds, src, wave, kt % S, kt + S, stride);
    tb_load_runs<DT, T>(lds + ((kt + 1) % S) * T::STAGE_BYTES, 0, wm, wn, lane, ra[0], rb[0]);
    mma_runs<DT, T, PRE, NB>(ra[last], rb[last], acc);
    chunk_hint<NB - PRE, NRD < NB - PRE ? NRD : NB - PRE, ISSUE ? T::DMA_PER_WAVE : 0>();
    __builtin_amdgcn_sched_barrier(0);
}

// Slice-ahead schedule, for wave tiles of few MFMAs: a transpose read takes
// so long that the schedule above, one K-chunk ahead, waits for it at every
// chunk. All operand runs of slice kt + 1 are read at once while slice kt's
// MFMAs run from registers; one wait + barrier per slice frees buffer kt % S
// (every wave holds slice kt in registers) and publishes slice kt + 1.
template <class T>
constexpr bool kTbAhead = 8 * (T::FM + T::FN) * T::KCH + T::FM * T::FN * T::NV <= 128;

// Wait with the copies of at most `slices` slices left in flight, barrier.
template <class T, int MAX>
__device__ __forceinline__ void tb_wait_slices(int slices) {
    if constexpr (MAX > 0) {
        if (slices >= MAX) return wait_vm_barrier<MAX * T::DMA_PER_WAVE>();
        tb_wait_slices<T, MAX - 1>(slices);
    } else {
        wait_vm_barrier<0>();
    }
}

template <int DT, class T, bool ISSUE>
__device__ __forceinline__ void tb_slice_ahead(uint8_t *lds, const uint8_t *const *src, long stride, int wave, int kt,
                                               int KT, int wm, int wn, int lane, const i32x4 (&ca)[T::KCH][T::FM],
                                               const i32x4 (&cb)[T::KCH][T::FN], i32x4 (&na)[T::KCH][T::FM],
                                               i32x4 (&nb)[T::KCH][T::FN],
                                               typename Acc<DT, 32>::type (&acc)[T::FM][T::FN]) {
    constexpr int S = T::STAGES;
    // a wait for the reads that the compiler knows of: with only the one in
    // the asm it would wait again, after the next reads
    __builtin_amdgcn_s_waitcnt(0xC07F);
    // in flight after the wait: slices kt + 2 .. kt + S - 1, or what is left
    if constexpr (ISSUE) wait_vm_barrier<(S - 2) * T::DMA_PER_WAVE>();
    else tb_wait_slices<T, S - 2>(KT - 2 - kt);
    __builtin_amdgcn_sched_barrier(0);
    const uint8_t *st = lds + ((kt + 1) % S) * T::STAGE_BYTES;
    // (after the last slice this reads a buffer nobody uses again; harmless)
#pragma unroll
    for (int kc = 0; kc < T::KCH; ++kc) tb_load_runs<DT, T>(st, kc, wm, wn, lane, na[kc], nb[kc]);
    if constexpr (ISSUE) tb_issue<DT, T>(lds, src, wave, kt % S, kt + S, stride);
#pragma unroll
    for (int kc = 0; kc < T::KCH; ++kc) mma_runs<DT, T, 0, T::FM * T::FN>(ca[kc], cb[kc], acc);
    __builtin_amdgcn_sched_barrier(0);
}

template <int DT, class T>
__device__ __forceinline__ void tb_accumulate_ahead(uint8_t *lds, const uint8_t *const *src, long stride, int wave,
                                                    int KT, int wm, int wn, int lane,
                                                    typename Acc<DT, 32>::type (&acc)[T::FM][T::FN]) {
    constexpr int S = T::STAGES;
    static_assert((S - 1) * T::DMA_PER_WAVE <= 63, "vmcnt range");
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < KT) tb_issue<DT, T>(lds, src, wave, s, s, stride);
    tb_wait_slices<T, S - 1>(KT - 1);
    i32x4 a0[T::KCH][T::FM], b0[T::KCH][T::FN], a1[T::KCH][T::FM], b1[T::KCH][T::FN];
#pragma unroll
    for (int kc = 0; kc < T::KCH; ++kc) tb_load_runs<DT, T>(lds, kc, wm, wn, lane, a0[kc], b0[kc]);
    int kt = 0;
    for (; kt + 1 + S < KT; kt += 2) {
        tb_slice_ahead<DT, T, true>(lds, src, stride, wave, kt, KT, wm, wn, lane, a0, b0, a1, b1, acc);
        tb_slice_ahead<DT, T, true>(lds, src, stride, wave, kt + 1, KT, wm, wn, lane, a1, b1, a0, b0, acc);
    }
    // at most one more slice issues a copy; then the rest
    if (kt + S < KT) tb_slice_ahead<DT, T, true>(lds, src, stride, wave, kt, KT, wm, wn, lane, a0, b0, a1, b1, acc);
    else tb_slice_ahead<DT, T, false>(lds, src, stride, wave, kt, KT, wm, wn, lane, a0, b0, a1, b1, acc);
    for (++kt; kt < KT; kt += 2) {
        tb_slice_ahead<DT, T, false>(lds, src, stride, wave, kt, KT, wm, wn, lane, a1, b1, a0, b0, acc);
        if (kt + 1 >= KT) break;
        tb_slice_ahead<DT, T, false>(lds, src, stride, wave, kt + 1, KT, wm, wn, lane, a0, b0, a1, b1, acc);
    }
}

// C = A * B with B(k, j) at element k * N + j. N a multiple of BN; K bytes
// per A row (Kb) a multiple of BKB.
template <int DT, class T>
__global__ __launch_bounds__(T::NTHREADS, 1) void tiled_gemm_tb(const uint8_t *__restrict__ A,
                                                               const uint8_t *__restrict__ B,
                                                               void *__restrict__ Cv, int M, int N,
                                                               int Kb, int tiles_m, int tiles_n,
                                                               EpiParams epi) {
    typedef TB<DT, T> P;
    typedef typename Acc<DT, 32>::type acc_t;
    constexpr int S = T::STAGES;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[T::LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    int tm, tn;
    tile_coords(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, T::GROUP_M, tm, tn);

    const uint8_t *src[T::DMA_PER_WAVE];
#pragma unroll
    for (int j = 0; j < T::DMA_PER_WAVE; ++j)
        src[j] = tb_src<DT, T>(A, B, M, N, Kb, tm, tn, wave * T::DMA_PER_WAVE + j, lane);
    // per-slice advance of B's units: BK rows
    const long stride = (long)P::BK * P::col_bytes(N);

    acc_t acc[T::FM][T::FN];
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j) acc[i][j] = acc_t{};

    const int KT = Kb / T::BKB;
    if constexpr (kTbAhead<T>) {
        tb_accumulate_ahead<DT, T>(lds, src, stride, wave, KT, wm, wn, lane, acc);
    } else {
#pragma unroll
        for (int s = 0; s < S; ++s)
            if (s < KT) tb_issue<DT, T>(lds, src, wave, s, s, stride);
        if (KT >= S) wait_vm_barrier<(S - 1) * T::DMA_PER_WAVE>();
        else wait_vm_barrier<0>();

        i32x4 ra[2][T::FM], rb[2][T::FN];
        tb_load_runs<DT, T>(lds, 0, wm, wn, lane, ra[0], rb[0]);
        int kt = 0;
        for (; kt + S < KT; ++kt) tb_slice<DT, T, true>(lds, src, stride, wave, kt, wm, wn, lane, ra, rb, acc);
        for (; kt < KT; ++kt) tb_slice<DT, T, false>(lds, src, stride, wave, kt, wm, wn, lane, ra, rb, acc);
    }

    const long row0 = (long)tm * T::BM + wm * T::WTM;
    const long col0 = (long)tn * T::BN + wn * T::WTN + (lane % 32);
    if constexpr (DT == S4)  // INT4 sums are carried times 256 (s4_lo_x16)
        epi_store_tile<DT, 32, T::FM, T::FN, T::NV, T::BM, T::BN, T::NTHREADS>(
            epi, Cv, acc, lds, (long)tm * T::BM, (long)tn * T::BN, row0, col0, lane / 32, M, N, ConvShift8());
    else
        epi_store_tile<DT, 32, T::FM, T::FN, T::NV, T::BM, T::BN, T::NTHREADS>(
            epi, Cv, acc, lds, (long)tm * T::BM, (long)tn * T::BN, row0, col0, lane / 32, M, N, ConvSame());
}

}  // namespace mpg
