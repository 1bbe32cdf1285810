// Row and column passes on lines of 768 points.
#define QPAT_LEN 768
#include "passes_inst.hpp"
