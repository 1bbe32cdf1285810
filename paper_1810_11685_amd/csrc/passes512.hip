// Row and column passes on lines of 512 points.
#define QPAT_LEN 512
#include "passes_inst.hpp"
