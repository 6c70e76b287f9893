// Row layout of the on-chip Lanczos kernel (resident.hip): a matrix small
// enough that one column of v_j fits in a workgroup's LDS.  Host only.
#pragma once

#include <cstdint>
#include <vector>

namespace vne {

// A workgroup of `waves` wavefronts owns every row; wave w takes `rounds`
// slices of 64 rows, and row (w * rounds + r) * 64 + lane is that lane's r-th
// row ("position").  Positions index v_j in LDS, so a lane's own rows are
// consecutive there; position `positions()` is a zero that padding entries
// read.  A slice is one of
//   empty  {0, 0, 0, 0}
//   short  {1, first, len, rows}: entries of lane l's row are the two 16-bit
//          positions of each words[(first + t) * 64 + l], t < len, len even
//          (rows of similar length share a slice: they are sorted by length)
//   long   {2, first, 0, rows}: lane l's row is spread over the wave: its
//          entries are words[(a + t) * 64 + lane], t < b, for every lane,
//          {a, b} = spans[2 * (first + l)], spans[2 * (first + l) + 1]
// Long rows (more than long_min entries) are dealt to the waves one by one:
// a hub would keep a single lane busy while the other waves are done.
// unit: every off-diagonal entry has the value off_value; words hold the
// off-diagonal entries only and diag the diagonal.  Otherwise words hold
// every entry and vals its value, two per word.
struct ResidentShape {
    int32_t waves = 0, rounds = 0;
    bool unit = false;
    double off_value = 0.0;
    int64_t word_rows = 0;               // 64 words each: one 64-lane read of v_j per half
    int32_t wave_long = 0;               // most long rows of a wave
    int64_t wave_tail = 0;               // most words of a wave's long rows past each row's first
    int32_t positions() const { return waves * rounds * 64; }
};

struct ResidentLayout : ResidentShape {
    std::vector<int32_t> slices;         // [waves * rounds][4]
    std::vector<uint32_t> words;
    std::vector<double> vals;            // [2 * words] or empty
    std::vector<int32_t> spans;
    std::vector<int32_t> row_of;         // [positions] row, or -1
    std::vector<double> diag;            // [positions] (unit) or empty
};

// Word rows of padding behind the last slice: the kernel loads the words of
// a slice in groups that may end past it.
constexpr int32_t kResidentSpareRows = 8;

// Most positions (they and the zero fit 16 bits).
constexpr int32_t kResidentMaxPositions = 65472;

// Most word rows, spare ones included: the kernel's byte offsets into the
// words (256 bytes a row) and the values (64 pairs a row) are 32-bit.  FP32
// matrices of unequal values reach it at about 1.07e9 entries.
constexpr int64_t resident_max_word_rows(bool unit, bool fp64) {
    return (int64_t(1) << 32) / (unit ? 256 : fp64 ? 64 * 16 : 64 * 8);
}

// The rows as a shape goes by them: their entries in words, the rows by falling
// length and how many of those are long.
struct ResidentRows {
    std::vector<int32_t> len, order;
    int64_t n_long = 0;
};

// What the layout of build_resident_layout looks like, without it; lay_out
// then makes it.
bool resident_shape(const int32_t *row_ptr, const int32_t *col, const double *val, int64_t n, int32_t waves,
                    int32_t max_rounds, bool fp64, ResidentShape *out, ResidentRows *rows);
void lay_out(const int32_t *row_ptr, const int32_t *col, const double *val, int64_t n, const ResidentShape &shape,
             const ResidentRows &rows, ResidentLayout *out);

// us of one on-chip step of a workgroup with `cols` columns.
double resident_step_us(const ResidentShape &s, int cols, bool fp64);

// Layout for `waves` wavefronts (1 .. 16) and vectors of the given type.
// Returns false when the rows need more than max_rounds rounds, or more word
// rows than resident_max_word_rows.
bool build_resident_layout(const int32_t *row_ptr, const int32_t *col, const double *val, int64_t n, int32_t waves,
                           int32_t max_rounds, ResidentLayout *out, bool fp64 = true);

}  // namespace vne
