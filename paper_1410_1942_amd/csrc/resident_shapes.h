// Shapes of the resident kernel, X(columns a thread, planes a column, keep,
// faces, workgroups a CU holds in batches), for its instances and the host's
// plan alike.  FP64 keeps q and the diagonal in registers up to 16 cells a
// thread, FP32 up to 32 (256 registers a thread with two waves a SIMD).
// Batches take the first shape marked that holds a grid (two workgroups a CU
// where its registers allow, which hide each other's exchanges).
#ifndef PCG_RESIDENT_SHAPES_H
#define PCG_RESIDENT_SHAPES_H

#define PCG_RESIDENT_FP64(X)                                                      \
    X(1, 1, true, false, 0)  X(1, 2, true, false, 0)  X(1, 3, true, false, 0)     \
    X(1, 4, true, false, 0)  X(2, 2, true, false, 0)  X(1, 6, true, false, 0)     \
    X(2, 4, true, false, 0)  X(1, 8, true, false, 1)  X(2, 6, true, false, 0)     \
    X(3, 4, true, false, 0)  X(2, 8, true, false, 1)  X(4, 4, true, false, 0)     \
    X(4, 6, false, false, 0) X(3, 8, false, false, 0) X(5, 6, false, false, 0)    \
    X(4, 8, false, false, 1)                                                      \
    X(1, 1, true, true, 0)   X(1, 2, true, true, 0)   X(1, 4, true, true, 0)      \
    X(2, 2, true, true, 0)   X(1, 6, true, true, 0)   X(2, 4, true, true, 0)      \
    X(1, 8, true, true, 0)   X(2, 5, true, true, 0)   X(3, 4, false, true, 0)     \
    X(2, 6, false, true, 0)

#define PCG_RESIDENT_FP32(X)                                                      \
    X(1, 1, true, false, 0)  X(1, 2, true, false, 0)  X(1, 3, true, false, 0)     \
    X(1, 4, true, false, 0)  X(2, 2, true, false, 0)  X(1, 6, true, false, 0)     \
    X(2, 4, true, false, 0)  X(1, 8, true, false, 2)  X(2, 6, true, false, 0)     \
    X(3, 4, true, false, 0)  X(4, 4, true, false, 0)  X(2, 8, true, false, 0)     \
    X(3, 8, true, false, 0)  X(4, 6, true, false, 0)  X(5, 6, true, false, 0)     \
    X(4, 8, true, false, 1)  X(6, 8, false, false, 1)                             \
    X(1, 1, true, true, 0)   X(1, 2, true, true, 0)   X(1, 4, true, true, 0)      \
    X(2, 2, true, true, 0)   X(2, 4, true, true, 0)   X(1, 8, true, true, 0)      \
    X(3, 4, true, true, 0)   X(2, 8, true, true, 0)   X(4, 4, true, true, 0)      \
    X(3, 6, true, true, 0)   X(5, 4, true, true, 0)   X(4, 6, false, true, 0)

#endif
