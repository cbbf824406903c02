// rve_solve_w8.hip -- the batched RVE solver compiled with 512-thread workgroups
// (eight wave64) into namespace fehmm::w8, for batches whose plans all keep their
// fronts in global memory.  Their tiles, sweeps and copies split over any number of
// waves, and one eight-wave workgroup per CU keeps half as many RVEs' fronts in the
// caches as two four-wave ones, with a shorter tail and, where the batch has fewer
// RVEs than the chip CUs, twice the waves per RVE (and no spills in the 128 x 128
// tiles: 64 instead of 128 accumulator registers per lane).  96 RVEs of 8^3 / 12^3 /
// 16^3: 1.32 s with four waves, 0.84-1.0 s with eight.
#define FEHMM_NWAVE 8
#define FEHMM_VARIANT w8
#include "rve_solve.hip"
