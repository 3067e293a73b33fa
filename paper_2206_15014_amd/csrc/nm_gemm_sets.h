// The patterns of one translation unit.  Kernels that are instantiated per pattern compile as one unit
// per set (NM_DMA_SET, given on the command line), so that the many instantiations build in parallel.
#ifndef NM_GEMM_SETS_H
#define NM_GEMM_SETS_H

#if NM_DMA_SET == 0
#define NM_SET_PATTERNS NM_CASE(2, 4, 8);
#elif NM_DMA_SET == 1
#define NM_SET_PATTERNS NM_CASE(1, 4, 8); NM_CASE(2, 4, 4);
#elif NM_DMA_SET == 2
#define NM_SET_PATTERNS NM_CASE(1, 4, 4); NM_CASE(1, 8, 8);
#elif NM_DMA_SET == 3
#define NM_SET_PATTERNS NM_CASE(2, 8, 8); NM_CASE(1, 8, 4);
#elif NM_DMA_SET == 4
#define NM_SET_PATTERNS NM_CASE(2, 8, 4);
#elif NM_DMA_SET == 5
#define NM_SET_PATTERNS NM_CASE(4, 4, 8); NM_CASE(4, 4, 4); NM_CASE(3, 4, 8);
#elif NM_DMA_SET == 6
#define NM_SET_PATTERNS NM_CASE(3, 4, 4); NM_CASE(4, 8, 8); NM_CASE(4, 8, 4);
#elif NM_DMA_SET == 7
#define NM_SET_PATTERNS NM_CASE(3, 8, 8); NM_CASE(3, 8, 4);
#elif NM_DMA_SET == 8
#define NM_SET_PATTERNS NM_CASE(5, 8, 8); NM_CASE(5, 8, 4);
#elif NM_DMA_SET == 9
#define NM_SET_PATTERNS NM_CASE(6, 8, 8); NM_CASE(6, 8, 4);
#elif NM_DMA_SET == 10
#define NM_SET_PATTERNS NM_CASE(7, 8, 8); NM_CASE(7, 8, 4);
#else
#error "NM_DMA_SET must be 0 .. 10"
#endif

// `name` with the number of this unit's set behind it
#define NM_SET_CAT2(a, b) a##b
#define NM_SET_CAT(a, b) NM_SET_CAT2(a, b)
#define NM_SET_NAME(name) NM_SET_CAT(name, NM_DMA_SET)

#endif
