// Included before every source that is compiled for the CPU: launches run their kernel on the emulated workgroups, or are
// only noted down by its name (emu_only_names).
#pragma once
#include "common.h"
#undef STS_LAUNCH
#define STS_LAUNCH(kernel, grid, block, shmem, stream, ...) \
  (emu::noted(#kernel) ? (void)0 : emu::run([&] { kernel(__VA_ARGS__); }, grid, block))
