// Host build of the two forms of the eigenvalue count in
// paper_2511_09798_amd/csrc/msvd.hpp, for CPU tests of one against the other.
#include <float.h>

#include "../../paper_2511_09798_amd/csrc/msvd.hpp"

extern "C" int count_pairs(const double* d2, const double* e2, int n, double x) {
    return mqh::msvd::negcount(d2, 1, e2, 1, n, x, DBL_MIN);
}
extern "C" int count_quotients(const double* d2, const double* e2, int n, double x) {
    return mqh::msvd::negcount_quotient(d2, 1, e2, 1, n, x, DBL_MIN);
}
// the same on the reversed sequences, read backwards
extern "C" int count_pairs_reversed(const double* d2, const double* e2, int n, double x) {
    return mqh::msvd::negcount(d2 + n - 1, -1, e2 + (n > 1 ? n - 2 : 0), -1, n, x, DBL_MIN);
}
