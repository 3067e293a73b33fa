/*
 * Test hook of libnm, not part of the ABI of include/nm.h: forces the tile variant that nm_gemm /
 * nm_gemm_q8 launch, so that the parity tests can cover every compiled variant whatever the
 * launcher would choose for a shape.  0 restores the automatic choice.  The value is one
 * process-wide atomic integer; a variant that cannot take a call hands it on to the next kernel
 * family as the automatic choice does.  Returns the previous value.
 */
#ifndef NM_TEST_HOOKS_H
#define NM_TEST_HOOKS_H
#include <stddef.h>
#ifdef __cplusplus
extern "C" {
#endif
int nm_test_force_gemm_tile(int cfg);

/*
 * Measurement hook of bench.py, not part of the ABI either: a register-resident loop of the
 * sparse integer MFMA that nm_gemm uses (v_smfmac_i32_16x16x128_i8, eight independent
 * accumulators per wavefront), `blocks` workgroups of four wavefronts, `iters` rounds of eight
 * instructions each - the instruction-issue ceiling of the matrix pipe with no memory traffic at
 * all.  counters_dev receives two 64-bit values from the first wavefront: shader clock cycles
 * and ticks of the constant 100 MHz clock spent in the loop (their ratio is the shader clock
 * under this load).  One launch executes blocks * 4 * iters * 8 instructions of
 * 2 * 16 * 16 * 128 dense-equivalent operations each.
 */
int nm_bench_smfmac_probe(int blocks, int iters, unsigned long long *counters_dev, void *hip_stream);

/*
 * Measurement hook of bench.py: the kernel variant that the most recent nm_gemm, nm_gemm_q8 or
 * nm_gemm_batch call of this process launched - the tile id of the LDS-direct kernels (>= 100),
 * 1 .. 3 for the register-staged kernel of the row layout, -1 for the kernel of the odd
 * shapes, 0 before the first call.  bench.py groups the launches of a step by it, as a kernel
 * trace groups them by kernel name.  One process-wide atomic integer: meaningful only while one
 * thread issues the calls.
 */
int nm_bench_last_gemm_tile(void);

/*
 * Test hook: how many launches nm_gemm would make of the kernel of the odd shapes for a call on its tiles,
 * the number of its output tiles, and the workgroups (of 256 threads) of the largest
 * launch.  Host arithmetic only.
 */
int nm_test_gemm_any_launches(int tokens, int K, int O, int N, int M, long long *tiles, unsigned *most_workgroups);

/*
 * Test hook: the tile id of the few-token kernels that nm_gemm would choose for one call in the
 * tiled layout, 0 where it would choose another family.  Host arithmetic only.
 */
int nm_test_few_tile(int tokens, int K, int O, int N, int M, int bits);

/*
 * Test hook: walks every load that the tiles of the kernel of the odd shapes would make for a call
 * and gives the ends of the bytes read (offsets of the last byte + 1) of X, vals and meta.  Returns 1,
 * 0 where the call would not go on tiles, or a negative status.  Host arithmetic only.
 */
int nm_test_gemm_any_reads(int tokens, int K, int ldx, int O, int N, int M, int bits, int layout,
                           size_t *x_end, size_t *v_end, size_t *m_end);

/*
 * Test hook: how many turns a workgroup of nm_project waits for the other workgroups of its scale group before it reads their values
 * itself; 0: it looks once.  Returns the previous value.  One process-wide atomic integer.
 */
int nm_test_project_patience(int turns);

/*
 * Test hook: the tile id that nm_gemm (out_dtype 3: nm_gemm_q8) would choose for one aligned call in the tiled layout, 0 where
 * another kernel family takes it, and where its tiles would start on their walk along K: the distance between neighbouring token
 * rows (upper 16 bits) and column tiles (lower 16) in K blocks of 128 columns (256 on tile 113), modulo their number.
 * Host arithmetic only, nothing is launched.
 */
int nm_test_gemm_plan(int tokens, int K, int O, int N, int M, int bits, int out_dtype, int *k_starts);

/* Test hook: the digest of the sources that the build made the library from, "unknown" where another way of compiling gave none. */
const char *nm_test_source_digest(void);
#ifdef __cplusplus
}
#endif
#endif
