// Row and column passes on lines of 32 points.
#define QPAT_LEN 32
#include "passes_inst.hpp"
