// Where the one-cell-per-wave kernels (rkc_wave.h) find a unit's pressure-dependent
// record.  Includes nothing, so that a host program can check the indices.
#pragma once

namespace rkcdev {

// The lane-group plan keeps records for the units from pd0 (the first of the round
// of SG lanes that holds a pressure-dependent one) to the last round's end; `count`
// of them are units.  The wave kernels' rounds are longer and their last one runs
// past that end.  -1: a unit without a record there.
constexpr int pdep_place(int unit, int pd0, int count) {
    return (unsigned)(unit - pd0) < (unsigned)count ? unit - pd0 : -1;
}

// Piece q (of 6) of the record at a place, in double2: interleaved by lane in rounds
// of SG.
constexpr int pdep_piece(int place, int q, int SG) {
    return (6 * (place / SG) + q) * SG + place % SG;
}

}  // namespace rkcdev
