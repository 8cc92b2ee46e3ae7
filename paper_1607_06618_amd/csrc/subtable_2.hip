// Table kernels for keys of 2 to 8 32-bit words.
#include "subtable.h"

namespace gerbil {

hipError_t sub_tables_2(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s) {
    switch (D) {
        GERBIL_SUB_CASE(2)
        GERBIL_SUB_CASE(3)
        GERBIL_SUB_CASE(4)
        GERBIL_SUB_CASE(5)
        GERBIL_SUB_CASE(6)
        GERBIL_SUB_CASE(7)
        GERBIL_SUB_CASE(8)
    }
    return hipErrorInvalidValue;
}

hipError_t launch_sub_tables(const CountArgs& a, const SubArgs& t, uint32_t block, uint32_t cus, hipStream_t s) {
    const uint32_t D = (a.k + 15) / 16, B = block;
    return D <= 8    ? sub_tables_2(a, t, D, B, cus, s)
           : D <= 14 ? sub_tables_9(a, t, D, B, cus, s)
           : D <= 19 ? sub_tables_15(a, t, D, B, cus, s)
           : D <= 25 ? sub_tables_20(a, t, D, B, cus, s)
                     : sub_tables_26(a, t, D, B, cus, s);
}

}  // namespace gerbil
