// Host build of the float64 fixed-point terms (gsdf_fixed.hpp), exposed
// through a C ABI for tests/test_magic_terms.py.
#define __host__
#define __device__
#include "../../paper_2111_13652_amd/csrc/gsdf_fixed.hpp"

extern "C" unsigned long long magic_term_host(double w, double x, int f) {
    const double magic = gsdf::magic_of(f);
    return gsdf::magic_term(std::fma(w, x, magic), 0ull - gsdf::double_bits(magic));
}
