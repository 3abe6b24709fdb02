// Check of the short binary32 sequences (exact_fp32.hpp) against the
// compiler's correctly rounded operators, over every float of a range.
#include "exact_fp32.hpp"
#include "tpc_internal.hpp"

namespace tpc {

namespace {

__device__ __forceinline__ bool same(float a, float b)
{
    return __float_as_uint(a) == __float_as_uint(b);
}

// the bit patterns lo, lo + 1, ..., hi - 1 as operand b
__global__ __launch_bounds__(kBlock) void k_check_exact(int op, uint32_t lo, uint32_t hi,
                                                        unsigned long long* __restrict__ bad)
{
    unsigned long long n = 0;
    for (uint64_t i = (uint64_t)lo + blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < hi;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const float b = __uint_as_float((uint32_t)i);
        if (op == 0) {
            n += !same(rcp_exact(b), 1.0f / b);
        } else if (op == 1) {
            n += !same(sqrt_exact(b), sqrtf(b));
        } else if (op == 2) {
            n += !same(rcp_any(b), 1.0f / b);
        } else {
            // eight numerators per denominator: a hash for the significand,
            // exponents spread over +-40, either sign
            const float r = rcp_exact(b);
            uint32_t h = (uint32_t)i * 2654435761u + 12345u;
            for (int k = 0; k < 8; ++k) {
                h ^= h >> 15;
                h = h * 2246822519u + 3266489917u * (uint32_t)k;
                const uint32_t e = 87u + (h >> 23) % 81u;
                const float a = __uint_as_float((h & 0x807FFFFFu) | (e << 23));
                n += !same(div_exact(a, b, r), a / b);
            }
        }
    }
    if (n) atomicAdd(bad, n);
}

}  // namespace

}  // namespace tpc

extern "C" int tpc_check_exact_fp32(int op, uint32_t lo, uint32_t hi, uint64_t* d_mismatches,
                                    void* stream)
{
    if (op < 0 || op > 3 || lo > hi || !d_mismatches) return TPC_ERR_INVALID_ARG;
    hipLaunchKernelGGL(tpc::k_check_exact, dim3(4096), dim3(tpc::kBlock), 0, (hipStream_t)stream,
                       op, lo, hi, (unsigned long long*)d_mismatches);
    return hipGetLastError() == hipSuccess ? TPC_OK : TPC_ERR_HIP;
}
