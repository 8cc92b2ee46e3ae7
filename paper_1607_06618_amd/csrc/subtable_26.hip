// Table kernels for keys of 26 to 30 32-bit words.
#include "subtable.h"

namespace gerbil {

hipError_t sub_tables_26(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s) {
    switch (D) {
        GERBIL_SUB_CASE(26)
        GERBIL_SUB_CASE(27)
        GERBIL_SUB_CASE(28)
        GERBIL_SUB_CASE(29)
        GERBIL_SUB_CASE(30)
    }
    return hipErrorInvalidValue;
}

}  // namespace gerbil
