// Which bytes of a slice's matrix the loads of consecutive rows into LDS touch (attn_single.hip).  Plain C++, so that the host can check it.
#pragma once

#if defined(__HIPCC__)
#define KVM_ROWS_FN __host__ __device__ __forceinline__
#else
#define KVM_ROWS_FN inline
#endif

namespace kvm {

// The rows from row0 on of a matrix of n rows: where they begin, and how many bytes there are from there to the end of the matrix.  A buffer
// load gets `begin` added to its base and `bytes` as its size, and no offset besides its lane's: the hardware compares a lane's offset with
// the size alone (a scalar offset of the instruction is not part of that comparison), and what lies beyond reads as zeros.
struct RowWindow { int begin, bytes; };
KVM_ROWS_FN constexpr RowWindow row_window(int n, int row0, int row_bytes) {
    return row0 < n ? RowWindow{row0 * row_bytes, (n - row0) * row_bytes} : RowWindow{n * row_bytes, 0};
}

// Load i of 64 lanes, 16 bytes each, of rows of `chunks` times 16 bytes: the row, counted from the window's first, that lane `lane` takes
// a chunk of, and where in that row.  Chunk ch of row r goes to position ch ^ r % 16 of the row's place in LDS.
KVM_ROWS_FN constexpr int row_of_lane(int i, int lane, int chunks) { return i * (64 / chunks) + lane / chunks; }
KVM_ROWS_FN constexpr int offset_in_row(int row, int lane, int chunks) { return ((lane % chunks) ^ (row & 15)) * 16; }

}  // namespace kvm
