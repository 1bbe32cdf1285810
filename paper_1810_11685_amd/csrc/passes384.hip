// Row and column passes on lines of 384 points.
#define QPAT_LEN 384
#include "passes_inst.hpp"
