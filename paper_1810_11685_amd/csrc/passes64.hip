// Row and column passes on lines of 64 points.
#define QPAT_LEN 64
#include "passes_inst.hpp"
