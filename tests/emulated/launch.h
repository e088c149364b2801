// Included before every source that is compiled for the CPU: launches run their kernel on the emulated workgroups.
#pragma once
#include "common.h"
#undef STS_LAUNCH
#define STS_LAUNCH(kernel, grid, block, shmem, stream, ...) emu::run([&] { kernel(__VA_ARGS__); }, grid, block)
