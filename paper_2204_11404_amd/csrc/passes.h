// Launches of the register passes.  Their kernels have many instantiations
// (unit kinds, chain lengths, precisions), compiled in parts of their own
// (passes.hip); the runtime in qecsv.hip calls them through these.
#pragma once

#include "kernels.hip"

namespace qec {

constexpr int kLaunchNoTable = 1;   // a dense unit without its Kraus table
constexpr int kLaunchNoFit = 2;     // the descriptor's layout does not fit a tile
constexpr int kLaunchNoKernel = 3;  // no instantiation for these units

template <typename T>
int launch_upass(const UnitPass& h, dim3 g, dim3 b, hipStream_t s, T* st, const UnitPass* pd,
                 const JobConst* jc, const BlockRT* rta, const BlockRT* rtb,
                 const Decision* da, Decision* db, double* part, int rev,
                 SlotStrides ss = SlotStrides{0, 0, 0}, const BlockDense* dna = nullptr,
                 const BlockDense* dnb = nullptr);

template <typename T>
int launch_spass(const UnitPass& h, bool redo, dim3 g, dim3 b, hipStream_t s, T* st, const UnitPass* pd,
                 const JobConst* jc, const BlockRT* rta, const BlockRT* rtb, const Decision* da,
                 Decision* db, double* part, int rev, SpecArgs sa, SlotStrides ss);

template <typename T>
int launch_flip(const FlipPass& h, int mode, bool keep, dim3 g, hipStream_t s, T* st, const FlipPass* pd,
                 const BlockRT* rta, const BlockRT* rtb, const Decision* da, Decision* db, double* part, int rev,
                 int n_cls_wg, bool per_tile, double* chunk_sums, SlotStrides ss);

}  // namespace qec
