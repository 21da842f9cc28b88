// Numeric refactorisation of G_x by dense fronts on the nodes of the tree
// plan (tree.h): part of the device Newton (newton.hip, kernels: fronts.hip).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "rh_internal.h"

namespace rh {

struct DevFronts;  // a network's fronts on the device

// Where the factorisation reads and writes (device memory).
struct FrontIo {
  const double *gx;  // values of G_x
  double *lu, *rinv, *stat;  // flat factors, pivot reciprocals; stat[2]: singular row + 1
};

// Builds the fronts; null in *out where the plan does not take the network.
// maps: the factors' flat layout and the entries of G_x in it.
rh_status fronts_build(const LuPlan &lu, const LuMaps &maps, DevFronts **out, std::string &err);
void fronts_free(DevFronts *f);
// P G_x P^T = L U into io.lu, on the null stream.
rh_status fronts_refactor(const DevFronts &f, const FrontIo &io, std::string &err);

}  // namespace rh
