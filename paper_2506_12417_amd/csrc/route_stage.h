// Where the prepared router's staging loads (route_packed_body, route_mfma.hip) read and write.  Plain C++, so that
// the host can check that every load stays inside its matrix.
//
// A stage holds the 64-term chunks stage * KSP ... + KSP - 1: for each, 32 token rows, then 32 * NB expert rows, every
// row one 128-byte line in eight 16-byte pieces, piece p of row r at position p ^ ((r / 2) & 7) (conflict-free
// fragment reads).  A load moves eight rows of a chunk (lane = row * 8 + position); a wavefront issues LPW of
// them per stage, XL of token rows and then WL of expert rows, the same in every stage but for a scalar offset.
#pragma once

template <int NB, int KSP>
struct RouteStage {
    static constexpr int TB = 32, EPT = 32 * NB, NWV = NB * KSP, CHUNK = 128;    // (bytes of a row's chunk)
    static constexpr int BYTES = (TB + EPT) * KSP * CHUNK;
    static constexpr int XL = (TB / 8 * KSP + NWV - 1) / NWV, WL = EPT / 8 * KSP / NWV, LPW = XL + WL;
    static_assert(EPT / 8 * KSP % NWV == 0 && (TB / 8 * KSP % NWV == 0 || XL == 1), "loads dealt to the wavefronts");

    static constexpr bool is_x(int i) { return i < XL; }
    static constexpr int slot(int wave, int i) { return wave + (i < XL ? i : i - XL) * NWV; }
    static constexpr int loads_of_chunk(int i) { return i < XL ? TB / 8 : EPT / 8; }
    static constexpr bool spare(int wave, int i) { return i < XL && slot(wave, i) >= TB / 8 * KSP; }   // more wavefronts than loads of token rows
    static constexpr int chunk(int wave, int i) { return slot(wave, i) / loads_of_chunk(i); }          // of the stage
    static constexpr int row(int wave, int i) { return slot(wave, i) % loads_of_chunk(i) * 8; }        // first row
    // its place in the stage
    static constexpr unsigned lds(int wave, int i) { return (unsigned)((chunk(wave, i) * (TB + EPT) + (i < XL ? 0 : TB) + row(wave, i)) * CHUNK); }
    // the per-lane offset in the matrix, for stage 0: a row past the matrix lies past the descriptor's range and reads zeros
    static constexpr unsigned lane_offset(int wave, int i, int lane, int d) {
        return (unsigned)(row(wave, i) + lane / 8) * (unsigned)d * 2u + (unsigned)(chunk(wave, i) * CHUNK) +
               (unsigned)((lane % 8 ^ (((i < XL ? 0 : TB) + row(wave, i) + lane / 8) >> 1 & 7)) << 4);
    }
    // The largest scalar offset at which the row still has this load's chunk.  Only the per-lane offset is
    // range-checked, so the scalar one stops here: chunks past the end (and stages past the last one) bring
    // earlier terms again.
    static constexpr unsigned last_offset(int wave, int i, int n_chunks) {
        return chunk(wave, i) < n_chunks ? (unsigned)((n_chunks - 1 - chunk(wave, i)) / KSP * KSP * CHUNK) : 0u;
    }
    static constexpr unsigned offset(int stage, unsigned last) {
        const unsigned at = (unsigned)stage * (unsigned)(KSP * CHUNK);
        return at < last ? at : last;
    }
};
