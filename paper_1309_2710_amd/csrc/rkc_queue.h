// The integrators' work queue: claims of cells by lane groups and waves.  Includes
// nothing, so that a host program that stands in for the lanes can compile it.
#pragma once

namespace rkcdev {

// The work queue is dealt out in QUEUE_PARTS parts: claim i of part q is position
// groups_total + i QUEUE_PARTS + q.  Claims on one address are served one by
// one, 11.4 ns each from anywhere on the chip (a single head held 262,144 cells
// of 10 evaluations to 1.75 ms, 16 to 1.06); 16 heads on lines of their own take
// 0.7 ns, and 64 measured the same.
constexpr int QUEUE_PARTS = 16, QUEUE_STRIDE = 32, QUEUE_INTS = QUEUE_PARTS * QUEUE_STRIDE;

// Claims on the work queue by groups of G lanes (64: one claim per wave; the
// NW waves that share a cell claim together).  A group claims from its own part
// until that is used up, then from the next; a part seen or claimed past its
// end is never asked again.
template <int G, int NW = 1>
struct Claim {
    int part, left;

    __device__ __forceinline__ void init() {
        // blocks and waves mixed: the first cells of waves with one number in
        // their block are alike in an ordered queue
        part = __builtin_amdgcn_readfirstlane(
            (int)((blockIdx.x + threadIdx.x / (64 * NW)) % QUEUE_PARTS));
        left = QUEUE_PARTS;
    }
    // unsigned: heads run past the end of the largest launches
    template <class P>
    __device__ __forceinline__ unsigned position(const P &p, int i) const {
        return (unsigned)(p.groups_total + part) + (unsigned)i * QUEUE_PARTS;
    }
    // the next position of the queue; n_cells once every part is used up.  A head
    // moves under other groups' claims, so lane 0 reads it for the whole group: lanes
    // that read it one by one may differ on where the part ends, and from then on
    // claim from different parts
    template <class P>
    __device__ __forceinline__ int next(const P &p, int g) {
        while (left > 0) {
            int i = 0;
            if (g == 0) i = atomicAdd(p.queue + part * QUEUE_STRIDE, 1);
            const unsigned pos = position(p, __shfl(i, 0, G));
            if (pos < (unsigned)p.n_cells) return (int)pos;
            for (;;) {
                part = (part + 1) % QUEUE_PARTS;
                if (--left == 0) break;
                if (g == 0)
                    i = __hip_atomic_load(p.queue + part * QUEUE_STRIDE, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                if (position(p, __shfl(i, 0, G)) < (unsigned)p.n_cells) break;
            }
        }
        return p.n_cells;
    }
};

}  // namespace rkcdev
