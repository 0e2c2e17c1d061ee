// The list bounds of the gather kernels, compiled for the host alone.
#include "../paper_1502_04993_amd/csrc/gather.h"

extern "C" unsigned gather_piece_end(unsigned e8, int end) { return glmr_gather::piece_end(e8, end); }
extern "C" int gather_cap() { return glmr_gather::CAP; }
extern "C" unsigned gather_entries() { return 8u * glmr_gather::ENTRIES; }
