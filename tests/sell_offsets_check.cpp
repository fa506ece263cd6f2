// The limit of the sliced-ELL layout counts a slice's entries, not the slots
// that fill up its last group of four (formats.cpp).
#include <cstdio>
#include <stdexcept>

#include "../paper_1204_2586_amd/csrc/host/setup.hpp"

using namespace auxp;

int main()
{
    // 69 slots per slice are stored as 72
    const std::vector<int64_t> off = sell_offsets(std::vector<int>(470000, 69), 64);
    if (off.size() != 470001 || off[1] != 72 * 64 || off.back() != (int64_t)470000 * 72 * 64) return 1;
    if (off.back() <= 0x7fffffff) return 2;
    try {
        sell_offsets(std::vector<int>(487000, 69), 64);
        return 3;
    } catch (const std::invalid_argument &) {
    }
    std::printf("OK\n");
    return 0;
}
