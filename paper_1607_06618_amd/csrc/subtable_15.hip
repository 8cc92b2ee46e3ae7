// Table kernels for keys of 15 to 19 32-bit words.
#include "subtable.h"

namespace gerbil {

hipError_t sub_tables_15(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s) {
    switch (D) {
        GERBIL_SUB_CASE(15)
        GERBIL_SUB_CASE(16)
        GERBIL_SUB_CASE(17)
        GERBIL_SUB_CASE(18)
        GERBIL_SUB_CASE(19)
    }
    return hipErrorInvalidValue;
}

}  // namespace gerbil
