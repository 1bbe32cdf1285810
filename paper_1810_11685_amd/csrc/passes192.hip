// Row and column passes on lines of 192 points.
#define QPAT_LEN 192
#include "passes_inst.hpp"
