// Numeric refactorisation of G_x by dense fronts on the nodes of the tree
// plan (tree.h): part of the device Newton (newton.hip, kernels: fronts.hip).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "rh_internal.h"

namespace rh {

struct DevFronts;  // a network's fronts on the device

// Device vectors of the Newton step.
struct FrontIo {
  const double *gx, *g;  // values of G_x; the mismatch
  double *lu, *stat;     // flat factors; stat[2]: singular row + 1
  double *x;             // the state
};

// Builds the fronts; null in *out where the plan does not take the network, or
// there is no memory for them.
// maps: the factors' flat layout and the entries of G_x in it.
rh_status fronts_build(const LuPlan &lu, const LuMaps &maps, DevFronts **out, std::string &err);
void fronts_free(DevFronts *f);
int64_t fronts_bytes(const DevFronts *f);  // of device memory (null: 0)
// All on the null stream: P G_x P^T = L U and L y = P g in the fronts;
// x -= G_x^{-1} g, from them; the factors out of the fronts into io.lu.
rh_status fronts_refactor(const DevFronts &f, const FrontIo &io, std::string &err);
rh_status fronts_solve(const DevFronts &f, const FrontIo &io, std::string &err);
rh_status fronts_factors(const DevFronts &f, const FrontIo &io, std::string &err);

}  // namespace rh
