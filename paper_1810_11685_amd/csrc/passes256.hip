// Row and column passes on lines of 256 points.
#define QPAT_LEN 256
#include "passes_inst.hpp"
