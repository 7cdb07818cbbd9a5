// aligned_pieces (csrc/row_pieces.h) against the addresses of a few rows.  Ends with status 1 at the first block that is
// wrong.
#include "row_pieces.h"

#include <cstdio>

int main()
{
    for (int eb = 2; eb <= 4; eb += 2)
        for (int co = 1; co <= 700; ++co)
            for (int extra = 0; extra <= 16; ++extra)  // a channel slice of a wider buffer
                for (int span = 64; span <= 512; span *= 2)
                    for (int first = 0; first < co; first += span) {
                        const int row = (co - first < span ? co - first : span) * eb, pitch = (co + extra) * eb;
                        for (int unit = 16; unit <= 64; unit *= 4)
                            for (int start = 0; start < 64; start += 16) {
                                bool aligned = row % unit == 0;
                                for (int r = 0; r < 8; ++r) aligned = aligned && (start + r * pitch + first * eb) % unit == 0;
                                if (rtoss::aligned_pieces(start, row, first * eb, pitch, unit) != aligned) {
                                    printf("%d channels from %d on, pitch %d bytes, unit %d\n", row / eb, first, pitch, unit);
                                    return 1;
                                }
                            }
                    }
    return 0;
}
