"""Columns of matrices of sixteen bins (or as many as the symbols hold) whose histograms take column tiles of more than one register
window, the last of which are not full: width in bits -> columns.  Bytes have a rule of their own."""

# rows read in place, or gathered from a matrix that the caches hold: tiles of two windows, and of four
TWO = {1: 1633, 2: 824, 3: 545, 4: 404, 5: 265, 6: 221, 7: 154, 9: 118, 10: 91, 11: 78, 12: 71, 13: 64, 14: 57, 15: 57, 16: 57}
FOUR = {6: 1881, 7: 851, 9: 235, 10: 191, 11: 164, 12: 141, 13: 127, 14: 113, 15: 113, 16: 113}
# gathered from a larger matrix: tiles of four windows
FOUR_GATHERED = {1: 201, 2: 201, 3: 201, 4: 193, 5: 145, 6: 121, 7: 103, 9: 79, 10: 73, 11: 67, 12: 61, 13: 55, 14: 49, 15: 49, 16: 49}
GATHERED_BYTES = 260_000_000
