// Row and column passes on lines of 96 points.
#define QPAT_LEN 96
#include "passes_inst.hpp"
