// Shapes of the table kernels specialised on (bits, K): the list that kmq_lut.hip (batch 1) and kmq_lut_columns.hip (batch
// columns side by side) instantiate, in this order.
#ifndef KMQ_LUT_SHAPES_H
#define KMQ_LUT_SHAPES_H

// ROW(bits, G, LPR, NWK, NWR, RS, waves per SIMD), one codebook per row; SC(...), block-scaled
#define KMQ_LUT_SHAPES(ROW, SC) \
    /* Several shapes may serve one (bits, K): lut_find takes the one whose grid comes out */ \
    /* most even over the CUs for the given N; the first listed wins ties. */ \
    /* 1-bit */                                              \
    ROW(1, 3, 16, 1, 4, 1, 4)      /* K = 1536, 16 rows per workgroup */ \
    ROW(1, 4, 16, 1, 4, 1, 4)      /* K = 2048, 16 rows per workgroup */ \
    ROW(1, 4, 16, 1, 2, 1, 4)      /* 8 */                   \
    ROW(1, 3, 32, 1, 4, 2, 4)      /* K = 3072, 16 */        \
    ROW(1, 3, 32, 1, 3, 3, 4)      /* 18 */                  \
    ROW(1, 3, 32, 1, 3, 2, 4)      /* 12 */                  \
    ROW(1, 4, 32, 1, 4, 2, 4)      /* K = 4096 */            \
    ROW(1, 3, 64, 1, 6, 2, 4)      /* K = 6144, 12 */        \
    ROW(1, 4, 64, 1, 4, 2, 4)      /* K = 8192,  8 */        \
    ROW(1, 4, 64, 1, 4, 3, 4)      /* 12 */                  \
    /* 2-bit */                                              \
    ROW(2, 3, 32, 1, 4, 2, 6)      /* K = 1536 */            \
    ROW(2, 4, 32, 1, 4, 2, 6)      /* K = 2048 */            \
    ROW(2, 3, 64, 1, 4, 2, 6)      /* K = 3072 */            \
    ROW(2, 4, 64, 1, 4, 2, 7)      /* K = 4096 */            \
    ROW(2, 3, 64, 2, 3, 2, 6)      /* K = 6144: two slices of 12-byte loads, 6 rows per workgroup */ \
    ROW(2, 4, 64, 2, 2, 4, 4)      /* K = 8192: 16 rows per workgroup (x, staged once per workgroup, is 16 KB here) */ \
    ROW(2, 4, 64, 2, 2, 2, 7)      /* 8 */                   \
    ROW(2, 4, 32, 7, 1, 4, 4)      /* K = 14336: 16-byte loads, 8 rows per workgroup (6.6 us on 4096 rows; 7.1 with 3 or 8 rows per wave) */ \
    ROW(2, 2, 64, 7, 1, 4, 7)      /* 8-byte loads, 4 rows per workgroup (7.05 us; taken for few rows) */ \
    /* 3-bit (lane slices are whole groups of three words = 32 elements) */ \
    ROW(3, 3, 16, 3, 1, 2, 6)      /* K = 1536: three slices of 12-byte loads, 8 rows per workgroup */ \
    ROW(3, 6, 32, 1, 4, 2, 6)      /* K = 2048 */            \
    ROW(3, 3, 32, 3, 1, 4, 6)      /* K = 3072: three slices of 12-byte loads (9216 rows: 5.2 us; 6.1 with one slice of 36-byte loads) */ \
    ROW(3, 6, 64, 1, 4, 2, 7)      /* K = 4096 (14336 rows: 7.7 us; 8.0 with 4 rows per wave) */ \
    ROW(3, 3, 64, 3, 2, 4, 6)      /* K = 6144: three slices of 12-byte loads, 8 rows per workgroup */ \
    ROW(3, 6, 64, 2, 2, 4, 4)      /* K = 8192: 16 rows per workgroup */ \
    ROW(3, 6, 64, 2, 2, 2, 6)      /* 8 */                   \
    ROW(3, 3, 64, 7, 1, 4, 6)      /* K = 14336: 12-byte loads, 4 rows per workgroup (4096 rows: 8.7 us; 9.0-9.2 with 24-byte loads) */ \
    /* 4-bit */                                              \
    ROW(4, 3, 64, 1, 4, 2, 6)      /* K = 1536: 12-byte loads */ \
    ROW(4, 4, 64, 1, 4, 2, 6)      /* K = 2048 */            \
    ROW(4, 3, 64, 2, 2, 2, 6)      /* K = 3072: two slices of 12-byte loads */ \
    ROW(4, 4, 64, 2, 2, 2, 6)      /* K = 4096 */            \
    ROW(4, 4, 64, 3, 2, 2, 6)      /* K = 6144 */            \
    ROW(4, 4, 64, 4, 1, 4, 4)      /* K = 8192: 4 rows per workgroup (4096 rows: 6.6 us; 7.0 with 2 or 6) */ \
    ROW(4, 4, 64, 4, 1, 2, 6)      /* 2 */                   \
    ROW(4, 4, 64, 7, 1, 4, 4)      /* K = 14336: 4 rows per workgroup (4096 rows: 10.5 us; 12.2 with 2, 10.9 with 6) */ \
    ROW(4, 4, 64, 7, 1, 2, 6)      /* 2 */                   \
    /* block-scaled format (lane slices of 32, 64 or 128 elements only) */ \
    SC(1, 4, 16, 1, 4, 1, 4)       /* K = 2048 */            \
    SC(1, 4, 16, 1, 2, 1, 4)                                 \
    SC(1, 4, 32, 1, 4, 2, 4)       /* K = 4096 */            \
    SC(1, 4, 64, 1, 4, 2, 4)       /* K = 8192 */            \
    SC(1, 4, 64, 1, 4, 3, 4)                                 \
    SC(2, 4, 32, 1, 4, 2, 6)       /* K = 2048 */            \
    SC(2, 4, 64, 1, 4, 2, 7)       /* K = 4096 */            \
    SC(2, 4, 64, 2, 2, 4, 4)       /* K = 8192 */            \
    SC(2, 4, 64, 2, 2, 2, 7)                                 \
    SC(2, 4, 32, 7, 1, 4, 4)       /* K = 14336 */           \
    SC(2, 2, 64, 7, 1, 4, 7)                                 \
    SC(3, 6, 32, 1, 4, 2, 6)       /* K = 2048 */            \
    SC(3, 6, 64, 1, 4, 2, 7)       /* K = 4096 */            \
    SC(3, 6, 64, 2, 2, 4, 4)       /* K = 8192 */            \
    SC(3, 6, 64, 2, 2, 2, 6)                                 \
    SC(3, 6, 32, 7, 1, 4, 4)       /* K = 14336 (lane slices of 64 elements: one block) */ \
    SC(4, 4, 64, 1, 4, 2, 6)       /* K = 2048 */            \
    SC(4, 4, 64, 2, 2, 2, 6)       /* K = 4096 */            \
    SC(4, 4, 64, 4, 2, 4, 4)       /* K = 8192: 8 rows per workgroup (8192 rows: 10.8 us; 11.3 with 4 rows, 12.8 with 16 rows and 16 waves) */ \
    SC(4, 4, 64, 4, 1, 4, 4)       /* 4 */                   \
    SC(4, 4, 64, 4, 1, 2, 6)                                 \
    SC(4, 4, 64, 7, 1, 4, 4)       /* K = 14336 */           \
    SC(4, 4, 64, 7, 1, 2, 6)

#endif
