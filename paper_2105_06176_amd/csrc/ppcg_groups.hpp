// ppcg_groups.hpp -- chunks that share their lists (see ppcg_stencil.hpp), on
// the host, from two hashes per chunk.
#pragma once

#include <algorithm>
#include <cstdint>
#include <map>
#include <utility>
#include <vector>

namespace ppcg {

// Four ints, as the device reads them.
struct GroupChunk {
    int list, mask, len, run;  // run: set on the device
};
struct GroupItem {
    int chunk, dst, masks, unused;  // copy this chunk's list (masks = 0) or its masks (1) to dst
};

struct ChunkGroups {
    std::vector<GroupChunk> chunk;
    std::vector<GroupItem> items;  // the representatives
    int64_t nlist = 0, nmask = 0;  // entries of the distinct lists and mask sets
    int longest = 0;
};

// One representative per hash and length: chunk c holds (cptr[c + 1] -
// cptr[c]) / height entries, its lists hash to hash[2 c], its masks to
// hash[2 c + 1].  With the length in the key a chunk never reads more entries
// than its representative has, also where two hashes agree by accident; equal
// hashes of equal length are compared on the device afterwards.
// false: the lists (12 bytes an entry) and masks (8) pass cap bytes.
inline bool group_chunks(int nchunks, int height, const int64_t *cptr, const unsigned long long *hash, int64_t cap,
                         ChunkGroups *out)
{
    using Key = std::pair<unsigned long long, int>;
    std::map<Key, int> lists, masks;
    ChunkGroups g;
    g.chunk.resize((size_t)nchunks);
    for (int c = 0; c < nchunks; ++c) {
        const int len = (int)((cptr[c + 1] - cptr[c]) / height);
        const auto l = lists.emplace(Key(hash[2 * (size_t)c], len), (int)g.nlist);
        const auto m = masks.emplace(Key(hash[2 * (size_t)c + 1], len), (int)g.nmask);
        if (l.second) {
            g.items.push_back({c, (int)g.nlist, 0, 0});
            g.nlist += len;
        }
        if (m.second) {
            g.items.push_back({c, (int)g.nmask, 1, 0});
            g.nmask += len;
        }
        if (12 * g.nlist + 8 * g.nmask > cap)
            return false;
        g.chunk[c] = {l.first->second, m.first->second, len, 0};
        g.longest = std::max(g.longest, len);
    }
    *out = std::move(g);
    return true;
}

}  // namespace ppcg
