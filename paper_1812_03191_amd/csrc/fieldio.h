// fieldio.h -- internal: a level's field to and from host memory.
#pragma once
#include <hip/hip_runtime.h>

#include "dfk.h"

namespace dfio {

// One entry count per dimension of the field (x fastest), its device array in
// the storage type (float with fp32) and the background added to, or taken
// off, each value.  Exactly one of out / in is set: count FP64 values, the
// caller's.  The copy is ordered on st and complete on return.
hipError_t field_io(hipStream_t st, const dfk::Geo &G, bool fp32, void *dev, const int e[3], double back,
                    double *out, const double *in);

// A run or engine that may use the staging buffers: they are freed with the
// last one.
struct User {
  User();
  ~User();
  User(const User &) = delete;
  User &operator=(const User &) = delete;
};

}  // namespace dfio
