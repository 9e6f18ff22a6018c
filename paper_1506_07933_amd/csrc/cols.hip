// cols.hip -- the kernels of cols.hpp, one per precision (lengths are data).
#include "cols.hpp"

namespace mifft {

const void* cols_kernel(bool fp64, bool mid)
{
    if (mid)
        return fp64 ? reinterpret_cast<const void*>(&k_cols_mid<double>)
                    : reinterpret_cast<const void*>(&k_cols_mid<float>);
    return fp64 ? reinterpret_cast<const void*>(&k_cols<double>) : reinterpret_cast<const void*>(&k_cols<float>);
}

hipError_t launch_cols(const ColsArgs<float>& a, dim3 grid, unsigned block, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL(k_cols<float>, grid, dim3(block), lds, s, a);
    return hipGetLastError();
}
hipError_t launch_cols(const ColsArgs<double>& a, dim3 grid, unsigned block, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL(k_cols<double>, grid, dim3(block), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_cols_mid(const MidArgs<float>& a, dim3 grid, unsigned block, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL(k_cols_mid<float>, grid, dim3(block), lds, s, a);
    return hipGetLastError();
}
hipError_t launch_cols_mid(const MidArgs<double>& a, dim3 grid, unsigned block, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL(k_cols_mid<double>, grid, dim3(block), lds, s, a);
    return hipGetLastError();
}

} // namespace mifft
