// The row variants (element type, metric, lanes per row, 16-byte pieces per lane) that kernels are built for.
#pragma once

// X(dtype, metric, G, NCH).  Float rows of 257 .. 512 and 513 .. 1024 bytes have variants of one and two pieces per
// lane: with the next larger ones (three and four pieces) up to three quarters of a gather step were empty pieces,
// and fewer rows were in flight (3 001 searches over 400-byte fp16 rows: 1.41 ms, now 0.79 ms).
#define ANN_ROW_VARIANTS(X)                                                  \
    X(kU8, kL2, 8, 1) X(kU8, kIP, 8, 1) X(kU8, kL2, 8, 2) X(kU8, kIP, 8, 2) X(kU8, kL2, 4, 2) X(kU8, kIP, 4, 2) \
    X(kF16, kL2, 8, 2) X(kF16, kIP, 8, 2) X(kF16, kL2, 32, 1) X(kF16, kIP, 32, 1) X(kF16, kL2, 32, 2) X(kF16, kIP, 32, 2) \
    X(kF16, kL2, 32, 3) X(kF16, kIP, 32, 3) X(kF32, kL2, 32, 1) X(kF32, kIP, 32, 1) X(kF32, kL2, 32, 2) X(kF32, kIP, 32, 2) \
    X(kF32, kL2, 8, 3) X(kF32, kIP, 8, 3) X(kF32, kL2, 32, 4) X(kF32, kIP, 32, 4)                               \
    X(kU8, kL2, 32, 3) X(kU8, kIP, 32, 3) X(kF16, kL2, 32, 6) X(kF16, kIP, 32, 6) X(kF32, kL2, 32, 12) X(kF32, kIP, 32, 12)
