#pragma once
#include <functional>
#include <string>
namespace emu {
// One block of nt work-items.  Wavefronts run as far as they can in the given
// order (waves: nt / 64 numbers), so the first one is a whole barrier interval
// ahead of the last.  Returns what was wrong, one line each: wavefronts waiting
// at different barriers, and words that two wavefronts touch between two
// barriers with a write among the accesses (needs code built with
// -fsanitize=thread, whose calls are answered by block_emu.cpp).
std::string run_block(int nt, const int *waves, const std::function<void()> &kernel);
}
