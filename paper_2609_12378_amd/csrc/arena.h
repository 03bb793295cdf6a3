// The scratch arena of a context: grow-only memory of the library's own, or a caller's workspace, which is never grown.
// The policy alone, the allocator being the caller's (context.hip: the HIP runtime).
#pragma once
#include <cstddef>
#include <cstdint>

struct Arena {
    void *base = nullptr;
    size_t bytes = 0;
    bool external = false;        // a caller's workspace (ckks_set_workspace)
    size_t refused = SIZE_MAX;    // the smallest size that the device has refused since the arena was last given back

    // a request of `need` bytes is known to fail
    bool refuses(size_t need) const { return need > bytes && (external || need >= refused); }

    void set(void *p, size_t n)
    {
        base = p;
        bytes = n;
        external = p != nullptr;
        refused = SIZE_MAX;
    }

    // room for `need` bytes; the library's own arena grows by giving the old one back first (rt.release, which waits
    // for its users) and asking for the new one (rt.allocate: null if there is no room)
    enum Status { OK, TOO_SMALL, NO_ROOM, RELEASE_FAILED };
    template <typename Runtime>
    Status take(size_t need, Runtime &rt)
    {
        if (need <= bytes) return OK;
        if (external) return TOO_SMALL;
        if (base) {
            if (!rt.release(base)) return RELEASE_FAILED;
            base = nullptr;
            bytes = 0;
        }
        const size_t size = (need + 255) & ~(size_t)255;
        base = rt.allocate(size);
        if (!base) {
            if (need < refused) refused = need;
            return NO_ROOM;
        }
        bytes = size;
        if (need >= refused) refused = SIZE_MAX;   // the device has the room again
        return OK;
    }
};

// Of a call that can run with g, g / 2, .. or 1 groups in need(g) bytes: the most groups whose request get(need(g)) is
// not refused (get returns false when it is), without asking for what the arena is known to refuse.  Asking costs the
// arena, a wait for the stream and two allocations, on every call of a program whose device has no room for g groups.
// 0: one group was refused as well.
template <typename Need, typename Get>
uint32_t most_groups(const Arena &a, uint32_t g, Need need, Get get)
{
    while (g > 1 && a.refuses(need(g))) g /= 2;
    while (!get(need(g))) {
        if (g == 1) return 0;
        g /= 2;
    }
    return g;
}
