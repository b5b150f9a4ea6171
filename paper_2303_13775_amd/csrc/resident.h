// Workgroups of 256 threads of a kernel that one compute unit holds at once, asked once per kernel.  The kernel is a
// template argument: keyed by its type, all kernels of one signature shared the answer of whichever was launched first,
// although their registers are cut for different residency (float pulls of 266k x 256 after a bf16 model in the same
// process 207 us, 170 without it and now).
#pragma once

#include <algorithm>

template <auto Kernel>
int resident_blocks() {
    static const int blocks = [] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, Kernel, 256, 0) != hipSuccess || nb < 1) nb = 4;
        return std::min(nb, 8);
    }();
    return blocks;
}
