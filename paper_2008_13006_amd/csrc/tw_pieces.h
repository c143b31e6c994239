/* Which 16-byte pieces of a matrix may be read whole.  Included by device code and, by itself, by a host test. */
#ifndef TW_PIECES_H_
#define TW_PIECES_H_

#if defined(__HIPCC__)
#define TW_HD __host__ __device__ __forceinline__
#else
#define TW_HD static inline
#endif

/* A matrix of rows x cols 16-bit elements, ld a multiple of 8, in a buffer that may end right behind its last element: the
 * number of rows (from the first) whose piece at column `col` (a multiple of 8) lies inside the buffer and holds something.
 * Behind a ragged row's end lies the row's pitch, which belongs to the buffer for every row but the last. */
TW_HD int tw_piece_rows(int col, int rows, int cols) {
    return col >= cols ? 0 : cols - col >= 8 ? rows : rows - 1;
}

#endif /* TW_PIECES_H_ */
