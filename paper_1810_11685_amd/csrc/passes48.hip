// Row and column passes on lines of 48 points.
#define QPAT_LEN 48
#include "passes_inst.hpp"
