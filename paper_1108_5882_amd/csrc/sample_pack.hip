// Rows of a device sample copied into the library's layout: the row stride
// changes from the caller's to the layout's and the padding columns are zeroed,
// in one pass.
#include "internal.hpp"

namespace pwa {
namespace {

constexpr int kPackThreads = 256;
constexpr int kPackUnits = 4096;    // 16-byte stores of one block's rows (about)

typedef unsigned long long u2 __attribute__((ext_vector_type(2)));

// Units of 8 bytes (an FP32 complex value, half an FP64 one): row r of dst
// takes width units of src and zeros up to dst_units (even), two units per
// thread and store.  Bound by HBM: every byte is read and written once, where a
// clear of the whole array followed by a pitched copy wrote the rows twice.
// 500,009 rows from 37 to 48 FP32 complex per row: 106 + 28 us before.
__global__ __launch_bounds__(kPackThreads) void pack_rows_kernel(unsigned long long *__restrict__ dst, int dst_units,
                                                                 const unsigned long long *__restrict__ src,
                                                                 int64_t src_units, int width, int64_t n,
                                                                 int rows_per_block) {
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const unsigned rows = (unsigned)(n - r0 < rows_per_block ? n - r0 : rows_per_block);
    const unsigned half = (unsigned)dst_units / 2, total = rows * half;
    const unsigned long long *s = src + r0 * src_units;
    u2 *d = reinterpret_cast<u2 *>(dst + r0 * dst_units);
    for (unsigned i = threadIdx.x; i < total; i += kPackThreads) {
        const unsigned r = i / half;
        const int c = 2 * (int)(i - r * half);
        const unsigned long long *p = s + r * src_units + c;
        u2 v = {0, 0};
        if (c < width) v.x = p[0];
        if (c + 1 < width) v.y = p[1];
        d[i] = v;
    }
}

}  // namespace

hipError_t launch_pack_rows(void *dst, size_t dst_pitch, const void *src, size_t src_pitch, size_t width, size_t n,
                            hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int dst_units = (int)(dst_pitch / 8);
    const int rows = std::max(1, 2 * kPackUnits / dst_units);
    hipLaunchKernelGGL(pack_rows_kernel, dim3((unsigned)((n + rows - 1) / rows)), dim3(kPackThreads), 0, stream,
                       static_cast<unsigned long long *>(dst), dst_units,
                       static_cast<const unsigned long long *>(src), (int64_t)(src_pitch / 8), (int)(width / 8),
                       (int64_t)n, rows);
    return hipGetLastError();
}

}  // namespace pwa
