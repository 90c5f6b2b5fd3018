// The streams' workspaces for split partial sums (host bookkeeping only).
#pragma once

namespace oc {

// A caller's streams and graphs are not seen to end, so what they leave behind
// is bounded: 2 GiB of 32 MiB workspaces.
constexpr int MAX_SPLIT_WORKSPACES = 64;

// One stream's workspaces: that of its eager calls, which run in order, and that
// of its last capture.  A captured call's graph may be replayed on any stream,
// beside eager calls and other graphs captured on this one, so each capture gets
// its own and keeps it (two instances of one graph share it, as they share the
// call's inputs and outputs).
// The allocator is asked once per stream and once per capture: one that found
// no memory, or MAX_SPLIT_WORKSPACES in use, stays without, so that all its calls
// take the same kernels.  `live` counts the process's workspaces.
struct SplitWorkspace {
    void *ptr = nullptr, *capture_ptr = nullptr;
    bool asked = false, captured = false;
    unsigned long long capture = 0;

    template <class Alloc>
    void *get(int &live, Alloc &&alloc) {
        if (!asked) {
            asked = true;
            ptr = make(live, alloc);
        }
        return ptr;
    }

    template <class Alloc>
    void *get_captured(int &live, unsigned long long id, Alloc &&alloc) {
        if (!captured || capture != id) {
            captured = true;
            capture = id;
            capture_ptr = make(live, alloc);
        }
        return capture_ptr;
    }

    // of the eager calls; a capture's stays with its graph
    template <class Free>
    void give_back(int &live, Free &&release) {
        if (!ptr) return;
        release(ptr);
        ptr = nullptr;
        --live;
    }

private:
    template <class Alloc>
    static void *make(int &live, Alloc &&alloc) {
        void *p = live < MAX_SPLIT_WORKSPACES ? alloc() : nullptr;
        if (p) ++live;
        return p;
    }
};

}  // namespace oc
