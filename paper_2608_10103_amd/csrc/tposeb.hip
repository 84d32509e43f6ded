// tposeb.hip - kernels outside the variant tables: B stored K x N row-major
// (tposeb_gemm.hpp), and rows of any length and alignment (ragged_gemm.hpp).
#include "variants.hpp"
#include "ragged_gemm.hpp"
#include "tposeb_gemm.hpp"

namespace mpg {

typedef TileCfg<256, 256, 2, 4, 128, 2, 4> Tb256;
typedef TileCfg<128, 128, 2, 4, 128, 4, 4> Tb128;
typedef TileCfg<64, 128, 2, 4, 128, 4, 4> Tb64x128;
typedef TileCfg<64, 64, 2, 2, 128, 4, 4> Tb64;

template <int DT, class T>
static TbKernel kernel() {
    typedef void (*fn_t)(const uint8_t *, const uint8_t *, void *, int, int, int, int, int, EpiParams);
    static const fn_t f = &tiled_gemm_tb<DT, T>;
    return TbKernel{reinterpret_cast<const void *>(f), T::BM, T::BN, T::NTHREADS};
}

template <int DT>
static TbKernel tb_pick(int tile) {
    switch (tile) {
        case TB_256: return kernel<DT, Tb256>();
        case TB_128: return kernel<DT, Tb128>();
        case TB_64X128: return kernel<DT, Tb64x128>();
        default: return kernel<DT, Tb64>();
    }
}

TbKernel tposeb_kernel(int dtype, int tile) {
    return dtype == F16 ? tb_pick<F16>(tile) : (dtype == S8 ? tb_pick<S8>(tile) : tb_pick<S4>(tile));
}

typedef TileCfg<64, 64, 2, 2, 128, 2, 4, 16> Ragged64;
typedef TileCfg<128, 128, 2, 4, 128, 2, 4> Ragged128;

template <int DT>
static RaggedKernel ragged_pick(int tile) {
    typedef void (*fn_t)(const uint8_t *, const uint8_t *, void *, int, int, int, int, int, EpiParams);
    // register sets: two for the small tile (FP16 16 x 4096 x 4100 18.8
    // against 26.1 us with one), one for the large (122 registers, so two
    // workgroups share a CU: FP16 3000^3 92.2 against 99.7 us with two)
    static const fn_t f64 = &ragged_gemm<DT, Ragged64, 2>, f128 = &ragged_gemm<DT, Ragged128, 1>;
    if (tile == 64)
        return RaggedKernel{reinterpret_cast<const void *>(f64), Ragged64::BM, Ragged64::BN, Ragged64::NTHREADS};
    return RaggedKernel{reinterpret_cast<const void *>(f128), Ragged128::BM, Ragged128::BN, Ragged128::NTHREADS};
}

RaggedKernel ragged_kernel(int dtype, int tile) {
    return dtype == F16 ? ragged_pick<F16>(tile) : (dtype == S8 ? ragged_pick<S8>(tile) : ragged_pick<S4>(tile));
}

}  // namespace mpg
