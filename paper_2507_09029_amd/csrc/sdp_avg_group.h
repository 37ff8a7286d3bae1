// Groups of 8 parameters that hold the end of one row and the start of the next: which 8 parameters a worker that trains only one of
// the two rows is asked for, so that nothing of the other is read.  Plain C++: the tests compile it for the host.
#pragma once

namespace sdp {

// Places from the group's first parameter to the first one that is read: none where the worker trains both rows, else to the last 8
// parameters of the first row, whose end the group's first `split` parameters are, or to the first 8 of the second.  Rows of 8
// parameters and more.
constexpr int group_shift(int split, bool first, bool second) { return first == second ? 0 : first ? split - 8 : split; }

// x: 8 parameters read `shift` places from the group's first -> the group's own, zeros in the place of those that were not read
constexpr void group_align(float (&x)[8], int shift) {
    const int n = shift < 0 ? -shift : shift;
    for (int s = 4; s > 0; s /= 2) {
        float y[8] = {};
        for (int i = 0; i < 8; ++i) {
            const float up = i >= s ? x[i - s] : 0.f, down = i + s < 8 ? x[i + s] : 0.f;
            y[i] = (n & s) == 0 ? x[i] : shift > 0 ? up : down;
        }
        for (int i = 0; i < 8; ++i) x[i] = y[i];
    }
}

} // namespace sdp
