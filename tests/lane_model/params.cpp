// The launch parameters, of which the kernels with segments and with a search
// per wavefront keep a copy in LDS, against the LDS that the plan leaves them.
#include <cstdio>

#include "mcs_layout.h"

int main() {
    std::printf("%zu\n", sizeof(mcs::SearchParams));
    return sizeof(mcs::SearchParams) > 256;
}
