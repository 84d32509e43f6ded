// ragged.hip - kernels for rows of any length and alignment (ragged_gemm.hpp).
#include "variants.hpp"
#include "ragged_gemm.hpp"

namespace mpg {

typedef TileCfg<64, 64, 2, 2, 128, 2, 4, 16> Ragged64;
typedef TileCfg<128, 128, 2, 4, 128, 2, 4> Ragged128;

template <int DT>
static RaggedKernel pick(int tile) {
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
    return dtype == F16 ? pick<F16>(tile) : (dtype == S8 ? pick<S8>(tile) : pick<S4>(tile));
}

}  // namespace mpg
