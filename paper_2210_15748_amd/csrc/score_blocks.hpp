// How many documents a workgroup of the mask-table kernels takes (host code, no HIP).
#pragma once
#include <stdint.h>

#include <algorithm>

namespace dessert {

// Documents per workgroup, docs_min to docs_max, so that the workgroups (gy for each block of documents) make whole rounds over the slots
// of an XCD, which takes every 8th block.  (Taken only where it is more than a halved block has: smaller ones 0.99 on average, up to 1.16.)
inline uint32_t whole_round_docs(uint64_t docs, uint64_t gy, uint64_t slots, uint64_t docs_max, uint32_t docs_min) {
    uint64_t rounds = ((docs + docs_max - 1) / docs_max * gy + 8 * slots - 1) / (8 * slots), most;
    while ((most = rounds * slots / gy * 8) == 0 || (docs + most - 1) / most > docs_max) ++rounds;
    return std::max((uint32_t)((docs + most - 1) / most), docs_min);
}

// Whether that is the faster choice, against a block of which code_bytes are read for table_bytes of masks.  What it brings are fewer
// tables to build, waves of documents more alike in length and a last round that is full; what it costs is that the workgroups of a
// block's query sets drift apart before the next block brings them together again, and then read its rows from memory each for itself.
// So not where the table is small against the rows, nor for sets of unequal numbers of chunks, whose long ones everything would wait for.
// Documents of one length gain nothing in the waves and lose what a block is short of a run of documents for every wave.
// 911 searches and scorings (14 L, C = 4 to 11, 1 to 250 sets of 1 to 300, 20 to 200 000 documents of 1 to 300 vectors) with whole
// rounds against blocks halved until there are 4096: time 0.93 on average, but more than 1.03 for 119 of them, up to 1.5 (3 sets of 118 x 62 662
// documents of 137, L = 64, C = 9 2.39 -> 3.60 ms).  By table_bytes / code_bytes, documents of one length: 0.02 to 0.15 1.04 to 1.08 on average, from 0.3
// on 0.82 (the kernel for any number of tables 0.95, but up to 1.2); of unequal length: the fixed-size kernel below 0.04 0.95 to 1.01, above 0.76 to
// 0.97; the other below 0.04 0.98 and up to 1.35, 0.04 to 0.08 0.94 and up to 1.13, above 0.90.  Where the rule says yes, 420 of them, 0.87 on average;
// of 6600 other calls 2 % take more than 1.03 of the time with halved blocks, at most 1.2.
inline bool whole_rounds_pay(uint64_t table_bytes, uint64_t code_bytes, bool equal_documents, bool equal_sets, bool any_tables) {
    if (!equal_sets || (equal_documents && any_tables)) return false;
    return table_bytes * 100 >= code_bytes * (equal_documents ? 30 : any_tables ? 8 : 4);
}

}  // namespace dessert
