// Far field between well separated drops by multipole and local expansions
// (expand.hip).  A context owns one Expand object; ehdbim.hip renews its plan
// for every new geometry and enqueues its kernels beside the direct sums.
#ifndef EHD_EXPAND_H
#define EHD_EXPAND_H

#include <hip/hip_runtime.h>

#include <vector>

namespace ehd {

constexpr int kExpClasses = 4;        // classes of expansion orders (M2L kernels)

// One drop as the expansions see it: far-field source slots, target nodes,
// centre, and the largest distances of both from the centre.
struct ExpandDrop {
    long long soff, ns, toff, nt;
    double c[3];
    double rs, rt;
};
// A translation work item: target drop, its pairs [first, last), which share
// of the source orders it takes (part of parts), output slot.
struct ExpandItem { int i, first, last, part, parts, slot; };
// A pair: source drop, expansion order, the target's centre from the
// source's in length units.
struct ExpandPair { int j, order; double D[3]; };

struct Expand {
    bool on = false;                  // some pairs of drops go through expansions
    int nd = 0;
    std::vector<unsigned char> near;  // [target drop][source drop]: 1 if summed directly
    double unit = 1.0;                // length unit, a power of two
    int nchunk = 1;                   // source chunks of the moments
    int nitems[kExpClasses] = {};
    int ntblocks = 0;                 // blocks of the evaluation, of 64 rowtiles targets
    int rowtiles = 1;

    // device buffers, kept from plan to plan and grown when needed
    struct Buf { void* p = nullptr; size_t cap = 0; };
    enum { DROPS, ORDERS, PAIRS, SLOTS, TBLOCKS, SCALE, MPART, MOM, LOCAL, COLS, ITEMS, LPART = ITEMS + kExpClasses,
           NBUF = LPART + kExpClasses };
    Buf buf[NBUF];
    template <typename T> T* at(int b) const { return static_cast<T*>(buf[b].p); }

    void release()
    {
        for (Buf& b : buf) {
            if (b.p) (void)hipFree(b.p);
            b = Buf{};
        }
        on = false;
    }
};

// Device memory of at least `bytes` in b (its content is lost when it grows).
hipError_t ensure(Expand::Buf& b, size_t bytes);

// Plan for the given drops: which pairs are expanded, to what order, and the
// work lists; on = false where the direct sums alone are expected to be
// faster or the device memory does not suffice.  Synchronous on `stream`.
hipError_t expand_plan(Expand& E, const std::vector<ExpandDrop>& drops, hipStream_t stream);

// Moments, translations and the evaluation at the targets for the kinds
// mask: out[9][T] receives the (unscaled) sums over the expanded pairs, the
// rows of the requested kinds only.  src: far-source records [14][Spad];
// tx, tn: target positions and normals [3][T].
hipError_t expand_enqueue(const Expand& E, hipStream_t stream, unsigned kinds, const double* src, long long Spad,
                          const double* tx, const double* tn, long long T, double* out);

}  // namespace ehd

#endif
