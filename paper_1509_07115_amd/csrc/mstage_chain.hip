// Moment stage for tiles of B = 32: the kernels and launches of the four-wave
// pipeline (mstage_chain.h), one item per workgroup.
#include "mstage_chain.h"

namespace dsbt {

namespace {

using namespace chain;

template <typename T, typename D, bool INV, bool KPH>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == sizeof(float) ? 2 : 1))) mstage_chain(const MItem* __restrict__ items, const void* src, void* dst,
                                                    PhaseArgs ph) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    T* lds = reinterpret_cast<T*>(lds_raw);
    const MItem& it = items[blockIdx.x];
    if (it.nch == 0) return;   // idle slot of the per-XCD schedule
    // Two workgroups on a compute unit place their waves on the SIMDs in the order
    // 0, 2, 1, 3, the second starting one SIMD further along, so that each SIMD
    // holds wave w of one and wave w - 1 of the other: this order of the roles pairs
    // every result wave with a pre or chain wave.
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (sizeof(T) == sizeof(float)) {
        if (it.NCB == 2) {
            run_item<T, D, INV, KPH, 2>(it, src, dst, ph, lds, wave);
            return;
        }
    }
    run_item<T, D, INV, KPH, 1>(it, src, dst, ph, lds, wave);   // FP64 items have one column block
}

// The operand table of one direction (kernels.h) from the FP64 blocks M_J[r][q] (row-major,
// R = 32 + k): workgroup (J, rb), thread = (group g, lane l).  The weight w_0 of odd l is
// folded into slot 0 of tile 0.
template <typename T>
__global__ void __launch_bounds__(256) pack_chain(const double* __restrict__ blocks, int k, int p, int inverse,
                                                  T* __restrict__ out) {
    const int J = blockIdx.x, rb = blockIdx.y, g = threadIdx.x >> 6, l = threadIdx.x & 63, R = 32 + k;
    const int row = 16 * rb + (l & 15);
    const double* M = blocks + (size_t)J * R * R;
    T* o = out + ((size_t)J * 4 + rb) * 1024 + 256 * g + 4 * l;
    for (int c = 0; c < 4; ++c) {
        const int col = 4 * (4 * g + c) + (l >> 4);
        double a = 0.0;
        if (row < R && col < R) {
            a = inverse ? M[(size_t)col * R + row] : M[(size_t)row * R + col];
            if (J == 0 && p == 0 && (inverse ? row : col) == 0) a *= 0.70710678118654752440;
        }
        o[c] = (T)a;
    }
}

}  // namespace

template <typename T>
hipError_t launch_pack_chain(const double* d_blocks, int k, int p, int NT, bool inverse, void* out, hipStream_t s) {
    if (k < 0 || k > 32 || NT < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(pack_chain<T>, dim3(NT, 4), dim3(256), 0, s, d_blocks, k, p, inverse ? 1 : 0,
                       static_cast<T*>(out));
    return hipGetLastError();
}

template <typename T>
size_t chain_lds_bytes(int ncb) {
    return sizeof(T) * (size_t)chain_lds_values(ncb > 1 ? 2 : 1);
}

template <typename T>
hipError_t set_lds_limits_chain() {
    hipError_t e = hipSuccess;
    const int bytes = (int)chain_lds_bytes<T>(sizeof(T) == sizeof(float) ? 2 : 1);
    auto set = [&](const void* f) {
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    };
    set((const void*)mstage_chain<T, float, true, false>);
    set((const void*)mstage_chain<T, float, true, true>);
    set((const void*)mstage_chain<T, float, false, false>);
    if constexpr (sizeof(T) == sizeof(double)) {
        set((const void*)mstage_chain<T, double, true, false>);
        set((const void*)mstage_chain<T, double, true, true>);
        set((const void*)mstage_chain<T, double, false, false>);
    }
    return e;
}

template <typename T, typename D>
hipError_t launch_mstage_chain(const MItem* d_items, int nitems, int ncb, const void* src, void* dst, bool inverse,
                               PhaseArgs ph, hipStream_t s) {
    if (nitems <= 0) return hipSuccess;
    if (!inverse && ph.use) return hipErrorInvalidValue;   // phases are applied to the inverse's input only
    if (sizeof(T) != sizeof(float) && ncb != 1) return hipErrorInvalidValue;
    if (sizeof(D) > sizeof(T)) return hipErrorInvalidValue;
    const size_t lds = chain_lds_bytes<T>(ncb);
    if (inverse && ph.use)
        hipLaunchKernelGGL((mstage_chain<T, D, true, true>), dim3(nitems), dim3(256), lds, s, d_items, src, dst, ph);
    else if (inverse)
        hipLaunchKernelGGL((mstage_chain<T, D, true, false>), dim3(nitems), dim3(256), lds, s, d_items, src, dst, ph);
    else
        hipLaunchKernelGGL((mstage_chain<T, D, false, false>), dim3(nitems), dim3(256), lds, s, d_items, src, dst, ph);
    return hipGetLastError();
}

template hipError_t launch_pack_chain<float>(const double*, int, int, int, bool, void*, hipStream_t);
template hipError_t launch_pack_chain<double>(const double*, int, int, int, bool, void*, hipStream_t);
template size_t chain_lds_bytes<float>(int);
template size_t chain_lds_bytes<double>(int);
template hipError_t set_lds_limits_chain<float>();
template hipError_t set_lds_limits_chain<double>();
template hipError_t launch_mstage_chain<float, float>(const MItem*, int, int, const void*, void*, bool, PhaseArgs,
                                                      hipStream_t);
template hipError_t launch_mstage_chain<double, float>(const MItem*, int, int, const void*, void*, bool, PhaseArgs,
                                                       hipStream_t);
template hipError_t launch_mstage_chain<double, double>(const MItem*, int, int, const void*, void*, bool, PhaseArgs,
                                                        hipStream_t);

}  // namespace dsbt
