// ppcg_pool.hpp -- releases of device memory, and the memory that a server
// keeps between its requests.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>
#include <shared_mutex>
#include <unordered_map>
#include <vector>

namespace ppcg {

// ---------------------------------------------------------------- releases
// Releasing device or pinned host memory synchronizes the whole device, and
// a device synchronization while another thread captures a graph invalidates
// that capture.  Every release in the library therefore holds this lock
// shared, and a graph capture holds it exclusively.
std::shared_mutex &release_mu();

// Device memory and streams that a server keeps between its requests.  hipFree
// waits for the whole device, so each of the 20 releases of a request's
// preparation waited for the iterations of the running ones (a burst of 12
// requests: 20.5 ms, with the pool 8.9).  A block is taken and given back by the threads that have
// called `use`; it is given back with no work pending on it (Use::stream, the
// one that a preparation works on, is synchronized first).
// The limit (a server's budget) bounds the blocks in use and the idle ones
// together: idle blocks are released before a new one passes it and whenever
// one is given back, and near it blocks are not rounded up to a size that
// others can reuse.  Only what is in use can pass it (see can_prepare in
// ppcg_serve.hip).  At most kMaxIdle stay idle; blocks above kMaxBlock
// are released when they are given back, all idle ones with the pool.
class DevPool {
  public:
    struct Use {
        DevPool *pool = nullptr;
        hipStream_t stream = nullptr;
        int64_t bytes = 0;  // taken less given back by this thread
    };
    static Use &use();  // this thread's
    ~DevPool();
    void set_limit(size_t bytes) { limit_ = bytes; }  // before the first block
    hipError_t take(void **p, size_t bytes);
    // NULL stream: none idle
    hipStream_t take_stream();
    bool give_stream(hipStream_t s);
    // of a block of some pool, by any thread; false: no pool's
    static bool give(void *p);

  private:
    static constexpr size_t kMaxBlock = (size_t)32 << 20, kMaxIdle = (size_t)256 << 20;
    static constexpr size_t kMaxStreams = 4;
    struct Block {
        DevPool *pool;
        size_t size;
        bool reusable;
    };
    static std::mutex &reg_mu();
    static std::unordered_map<void *, Block> &reg();  // blocks of all pools
    void trim(size_t most);  // idle bytes, at most kMaxIdle and what the limit leaves
    std::mutex mu_;
    std::multimap<size_t, void *> idle_;
    size_t idle_bytes_ = 0, out_ = 0, limit_ = (size_t)-1;
    std::vector<hipStream_t> streams_;
};

}  // namespace ppcg
