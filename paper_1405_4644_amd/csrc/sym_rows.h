// Which elements of a symmetric matrix given by its lower triangle stand for
// the rows i, i + 1 of column j of a block of its product: i even, 32 x 32
// blocks, the block on the diagonal (diag) or below it, end: the last one of
// the diagonal.  Rows past the matrix and above the diagonal stand for zeros,
// but are loaded from somewhere as the others are: always from the lower
// triangle.
#pragma once

// first row of the 16-byte load of both (not for end: there each row has a
// load of its own, sym_row), c the column, or the last one if that is past it
constexpr int sym_first(int i, int c, int n, bool diag)
{
    const int last = n - 2;  // (a matrix with more than one block)
    return diag ? (i > c ? i : c) : (i < last ? i : last);
}
constexpr int sym_row(int i, int c, int n)
{
    const int r = i > c ? i : c;
    return r < n - 1 ? r : n - 1;
}
// the loaded values v0, v1 as those of rows i and i + 1, the diagonal halved
constexpr double sym_even(double v0, double v1, int i, int j, int n, bool end)
{
    const double x = (end || i + 1 < n) ? v0 : v1;
    return (i < n && i >= j) ? (i == j ? 0.5 * x : x) : 0.0;
}
constexpr double sym_odd(double v0, double v1, int i, int j, int n, bool diag, bool end)
{
    const double y = (diag && !end && i + 1 == j) ? v0 : v1;
    return (i + 1 < n && i + 1 >= j) ? (i + 1 == j ? 0.5 * y : y) : 0.0;
}
