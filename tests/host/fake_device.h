// What the host stand-in of the evaluation saw (fake_device.cpp), for the driver.
#pragma once

#include <cstdint>

namespace ks {
struct EvalSeen {
  bool uniq;        // the different records are evaluated
  uint32_t mask;    // of these families
  bool pair;        // with per-pair outputs
  bool apart;       // no two regions it may write overlap
};
extern EvalSeen eval_seen;
}  // namespace ks
