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
            // sixteen numerators per denominator: a hash for the significand,
            // exponents over +-40 and over +-80, either sign; op 4: the
            // special values too
            const float r = rcp_exact(b);
            uint32_t h = (uint32_t)i * 2654435761u + 12345u;
            for (int k = 0; k < 16; ++k) {
                h ^= h >> 15;
                h = h * 2246822519u + 3266489917u * (uint32_t)k;
                const uint32_t e = k < 8 ? 87u + (h >> 23) % 81u : 47u + (h >> 23) % 160u;
                const float a = __uint_as_float((h & 0x807FFFFFu) | (e << 23));
                n += !same(op == 3 ? div_exact(a, b, r) : div_exact_special(a, b, r), a / b);
            }
            if (op == 4)
                for (uint32_t k = 0; k < 6; ++k) {
                    // +-0, +-infinity, NaN of either sign (any NaN for NaN)
                    const float a = __uint_as_float((k & 1u) << 31 | (k < 2 ? 0u : k < 4 ? 0x7F800000u : 0x7FC00000u));
                    const float q = div_exact_special(a, b, r);
                    n += !(same(q, a / b) || (q != q && a != a));
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
    if (op < 0 || op > 4 || lo > hi || !d_mismatches) return TPC_ERR_INVALID_ARG;
    hipLaunchKernelGGL(tpc::k_check_exact, dim3(4096), dim3(tpc::kBlock), 0, (hipStream_t)stream,
                       op, lo, hi, (unsigned long long*)d_mismatches);
    return hipGetLastError() == hipSuccess ? TPC_OK : TPC_ERR_HIP;
}
