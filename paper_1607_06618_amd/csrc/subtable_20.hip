// Table kernels for keys of 20 to 25 32-bit words.
#include "subtable.h"

namespace gerbil {

hipError_t sub_tables_20(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s) {
    switch (D) {
        GERBIL_SUB_CASE(20)
        GERBIL_SUB_CASE(21)
        GERBIL_SUB_CASE(22)
        GERBIL_SUB_CASE(23)
        GERBIL_SUB_CASE(24)
        GERBIL_SUB_CASE(25)
    }
    return hipErrorInvalidValue;
}

}  // namespace gerbil
