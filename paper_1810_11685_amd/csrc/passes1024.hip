// Row and column passes on lines of 1024 points.
#define QPAT_LEN 1024
#include "passes_inst.hpp"
