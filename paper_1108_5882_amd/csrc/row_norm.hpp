// The sum of |A_a|^2 over one lane's share of a row of k complex values, eight lanes
// per row: lane sub takes the pairs of columns 2 c and 2 c + 1 with c = sub, sub + 8,
// ... in order.  Which values a lane may read depends on the row length: rows of an
// even number of columns start on 16 bytes and hold both columns of every pair, so
// two(c) reads columns 2 c and 2 c + 1 at once.  Layouts of one and three columns
// exist (k = 1 and 3): there the pair of the last column would start on 8 bytes and
// end past the row, past the sample in its last row, and one(a) reads column a alone.
#pragma once

namespace pwa {

template <typename Two, typename One>
__host__ __device__ inline double row_norm_share(int k, bool even_rows, int sub, Two two, One one) {
    double s = 0.0;
    for (int c = sub; 2 * c < k; c += 8) {
        if (even_rows) {
            const auto v = two(c);
            s += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
            if (2 * c + 1 < k) s += (double)v.z * (double)v.z + (double)v.w * (double)v.w;
        } else {
            const auto v = one(2 * c);
            s += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
            if (2 * c + 1 < k) {
                const auto u = one(2 * c + 1);
                s += (double)u.x * (double)u.x + (double)u.y * (double)u.y;
            }
        }
    }
    return s;
}

}  // namespace pwa
