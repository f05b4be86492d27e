// The redundancy stream's exchange of the streamed rows' weights within a wave: 16 lanes hold the weights of row `r` and of
// row `r + 16` of a stage, every lane reads back those of its accumulator's rows.  Plain C++, so that its indexes can be
// checked without a GPU.
#pragma once

namespace ems {

struct RedWeights {
    static constexpr int kLanes = 64, kRows = 32;          // kRows: rows per stage
    static constexpr int kSecond = 16;                     // a lane's second weight lies this far behind its first
    // behind the rows: where the lanes that hold none write, so that the stores need no condition (both of them)
    static constexpr int kFloats = kRows + kLanes + kSecond;

    // Lane l holds accumulator rows 4 (l / 16) .. + 3 of column l % 16: the tile's diagonal where the column is among them.
    static constexpr bool holds(int lane) { return lane / 16 == lane % 16 / 4; }
    // where a lane writes its first weight: the place of its row, or one that nobody reads
    static constexpr int slot(int lane) { return holds(lane) ? lane % 16 : kRows + lane; }

    // every store lies in the kFloats of its stage, every row is written once, and no other lane writes to a row's place
    static constexpr bool sound()
    {
        for (int row = 0; row < kRows; ++row) {
            int writers = 0;
            for (int lane = 0; lane < kLanes; ++lane) writers += (slot(lane) == row) + (slot(lane) + kSecond == row);
            if (writers != 1) return false;
        }
        for (int lane = 0; lane < kLanes; ++lane)
            if (slot(lane) < 0 || slot(lane) + kSecond >= kFloats) return false;
        return true;
    }
};

}  // namespace ems
