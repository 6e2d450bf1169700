// block_table.hpp -- blocks by position on the host: packed keys and a flat
// hash table from key to block number.  Planning a mesh makes 7 to 30 lookups
// per block; in a table of one array with linear probing each costs a few ns,
// in a node-based map a cache miss and, when it is filled, an allocation
// (regrid decision of 2304 blocks 0.83 -> 0.2 ms, their plan 0.52 -> 0.35 ms,
// on one host).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace agile {

// (level, x, y, z) in sorted order; level 1 to 15, coordinates below 2^20
inline uint64_t block_key(int level, int64_t x, int64_t y, int64_t z) {
    return (uint64_t(level) << 60) | (uint64_t(x) << 40) | (uint64_t(y) << 20) | uint64_t(z);
}

class BlockTable {
public:
    // room for n keys at a load of at most one half
    explicit BlockTable(size_t n) {
        int bits = 4;
        while ((size_t(1) << bits) < 2 * n) ++bits;
        slot_.assign(size_t(1) << bits, Slot{0, -1});
        shift_ = 64 - bits;
        mask_ = slot_.size() - 1;
    }
    // false when the key is there already
    bool insert(uint64_t key, int value) {
        size_t i = place(key);
        if (slot_[i].key == key) return false;
        slot_[i] = Slot{key, value};
        return true;
    }
    int find(uint64_t key) const { return slot_[place(key)].value; }   // -1: none

private:
    struct Slot {
        uint64_t key;   // 0: free (the level of a block is at least 1)
        int value;
    };
    size_t place(uint64_t key) const {
        // one product spreads boxes of blocks evenly (1.1 probes per block of a
        // 16^3 box; a full mix of the bits takes 1.5)
        size_t i = size_t((key * 0x9e3779b97f4a7c15ULL) >> shift_);
        while (slot_[i].key != 0 && slot_[i].key != key) i = (i + 1) & mask_;
        return i;
    }
    std::vector<Slot> slot_;
    size_t mask_;
    int shift_;
};

} // namespace agile
