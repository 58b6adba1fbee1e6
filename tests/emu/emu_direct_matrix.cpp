// emu_direct.cpp with the matrix path: same program, same usage.
#include "emu_matrix.h"

#include "emu_direct.cpp"
