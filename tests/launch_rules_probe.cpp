// Test-only: the library's launch rules, which its C ABI does not show, for a plan handle
// (tests/test_launch_rules.py links this to libemu.so).
#include "emu.h"
#include "emu_internal.h"

extern "C" void probe_reshard(const void* plan, uint32_t groups, int32_t* out) {
  const emu::LaunchRule r = emu::reshard_rule(*static_cast<const emu::Plan*>(plan), groups);
  out[0] = r.policy;
  out[1] = r.cap;
  out[2] = r.blocks;
}

extern "C" void probe_bucket(const void* plan, int32_t side, uint64_t B, int32_t unpack, int32_t* out) {
  const emu::LaunchRule r = emu::bucket_rule(static_cast<const emu::Plan*>(plan)->side[side], B, unpack != 0);
  out[0] = r.policy;
  out[1] = r.cap;
}
