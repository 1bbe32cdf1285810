// Row and column passes on lines of 128 points.
#define QPAT_LEN 128
#include "passes_inst.hpp"
