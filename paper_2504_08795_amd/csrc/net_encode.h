// A network's plan as launches (host logic, no GPU needed).
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "kernels.h"
#include "net_plan.h"

namespace daris {

struct LaunchRt {
  KernelLaunch kl;
  const void* dev = nullptr;  // the launch's argument block inside the task's device buffer
  double flops = 0;           // arithmetic of the layer(s) a dense-convolution launch computes, else 0
};

// A whole network as launches in execution order, encoded at registration; layer l issues launches [layer_lo[l],
// layer_lo[l + 1]) (none for the earlier member of a launch pair).
struct LaunchSeq {
  std::vector<LaunchRt> launches;
  std::vector<int> layer_lo;
  int in_launch = -1, out_launch = -1;  // the launches that read the job's input / write its logits
  uint32_t in_off = 0, out_off = 0;     // byte offset of that pointer inside the argument block
};

// Encodes the whole network as launches in execution order, with its activation tensors in `slots` (one device
// buffer per slot of the plan) and its split-K partial sums in `ws`; the weights must be on the device.  The two pointers
// that change from job to job (the input of the first launch, the logits of the last) stay null in the argument blocks.
// wave_prio: ConvArgs::wave_prio.  Returns "" or an error text.
std::string encode_network(const NetPlan& net, bool wave_prio, const KernelTable& kt, const JoinedTable& joined, const std::vector<void*>& slots, float* ws, LaunchSeq* seq);

}  // namespace daris
