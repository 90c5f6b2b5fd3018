// One stream's workspace for split partial sums (host bookkeeping only).
#pragma once

namespace oc {

// Asked of the allocator once: a stream whose first call found no memory stays
// without a workspace, so that no later call allocates and all of a stream's
// calls take the same kernels.
struct SplitWorkspace {
    void *ptr = nullptr;
    bool asked = false;

    template <class Alloc>
    void *get(Alloc &&alloc) {
        if (!asked) {
            asked = true;
            ptr = alloc();
        }
        return ptr;
    }
};

}  // namespace oc
