// Batch items run as register tile passes (batch_tile.hip).
#pragma once

#include <vector>

#include "circuit.h"
#include "observable.h"

namespace qsv {

struct BatchTileItem {
  const qsv_circuit* c;
  const qsv_observable* o;
  int index, theta_off, grad_off;  // energy, first parameter, first gradient entry
};

struct BatchTiles;

// Whether an item of this circuit can run as tile passes.
bool batch_tiles_take(const qsv_circuit& c);

// Plans the items and allocates and fills what they need on the device. Items
// whose circuit turns out not to be plannable are returned in left. *out stays
// null when none is taken.
template <typename R>
int batch_tiles_build(const std::vector<BatchTileItem>& items, BatchTiles** out, std::vector<BatchTileItem>& left);

// Enqueues one evaluation (kernels only: it can be captured).
template <typename R>
int batch_tiles_launch(const BatchTiles* t, const double* theta, double* energies, double* grads, hipStream_t st);

void batch_tiles_free(BatchTiles* t);

}  // namespace qsv
