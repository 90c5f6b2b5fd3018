// The streams' workspaces for split partial sums (host bookkeeping only).
#pragma once

namespace oc {

// A caller's streams are not seen to end, so what they leave behind is bounded:
// 2 GiB of 32 MiB workspaces.
constexpr int MAX_SPLIT_WORKSPACES = 64;

// One stream's workspace, asked of the allocator once: a stream whose first
// call found no memory, or MAX_SPLIT_WORKSPACES in use, stays without one, so
// that no later call allocates and all of a stream's calls take the same
// kernels.  `live` counts the process's workspaces.
struct SplitWorkspace {
    void *ptr = nullptr;
    bool asked = false;

    template <class Alloc>
    void *get(int &live, Alloc &&alloc) {
        if (!asked) {
            asked = true;
            if (live < MAX_SPLIT_WORKSPACES) ptr = alloc();
            if (ptr) ++live;
        }
        return ptr;
    }

    template <class Free>
    void give_back(int &live, Free &&release) {
        if (!ptr) return;
        release(ptr);
        ptr = nullptr;
        --live;
    }
};

}  // namespace oc
