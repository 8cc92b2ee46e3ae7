// Table kernels for keys of 9 to 14 32-bit words.
#include "subtable.h"

namespace gerbil {

hipError_t sub_tables_9(const CountArgs& a, const SubArgs& t, uint32_t D, uint32_t B, uint32_t cus, hipStream_t s) {
    switch (D) {
        GERBIL_SUB_CASE(9)
        GERBIL_SUB_CASE(10)
        GERBIL_SUB_CASE(11)
        GERBIL_SUB_CASE(12)
        GERBIL_SUB_CASE(13)
        GERBIL_SUB_CASE(14)
    }
    return hipErrorInvalidValue;
}

}  // namespace gerbil
