// ppcg_pool.hip -- DevPool (host code; see ppcg_pool.hpp).

#include "ppcg_pool.hpp"

#include <algorithm>
#include <iterator>

namespace ppcg {

std::shared_mutex &release_mu()
{
    static std::shared_mutex m;
    return m;
}

DevPool::Use &DevPool::use()
{
    static thread_local Use u;
    return u;
}

std::mutex &DevPool::reg_mu()
{
    static std::mutex m;
    return m;
}

std::unordered_map<void *, DevPool::Block> &DevPool::reg()
{
    static std::unordered_map<void *, Block> r;
    return r;
}

DevPool::~DevPool()
{
    trim(0);
    for (hipStream_t s : streams_)
        (void)hipStreamDestroy(s);
    std::lock_guard<std::mutex> lk(reg_mu());
    for (auto it = reg().begin(); it != reg().end();)  // (blocks still out are released by hipFree)
        it = it->second.pool == this ? reg().erase(it) : std::next(it);
}

hipError_t DevPool::take(void **p, size_t bytes)
{
    size_t size = 512;  // powers of two and the three sizes between them
    while (size < bytes)
        size *= 2;
    if (size > 2048)
        for (int q = 5; q < 8; ++q)
            if (size / 8 * q >= bytes) {
                size = size / 8 * q;
                break;
            }
    bool reusable = size <= kMaxBlock;
    {
        std::lock_guard<std::mutex> lk(mu_);
        auto it = reusable ? idle_.find(size) : idle_.end();
        if (it != idle_.end()) {
            *p = it->second;
            idle_.erase(it);
            idle_bytes_ -= size;
            out_ += size;
            use().bytes += (int64_t)size;
            return hipSuccess;
        }
        if (!reusable || out_ >= limit_ || size > limit_ - out_) {
            size = std::max<size_t>(bytes, 256);
            reusable = false;
        }
        out_ += size;
    }
    trim(kMaxIdle);
    hipError_t e = hipMalloc(p, size);
    if (e == hipErrorOutOfMemory) {
        trim(0);
        (void)hipGetLastError();
        e = hipMalloc(p, size);
    }
    if (e != hipSuccess) {
        std::lock_guard<std::mutex> lk(mu_);
        out_ -= size;
        return e;
    }
    use().bytes += (int64_t)size;
    std::lock_guard<std::mutex> lk(reg_mu());
    reg()[*p] = {this, size, reusable};
    return hipSuccess;
}

bool DevPool::give(void *p)
{
    Block b;
    {
        std::lock_guard<std::mutex> lk(reg_mu());
        auto it = reg().find(p);
        if (it == reg().end())
            return false;
        b = it->second;
        if (!b.reusable)
            reg().erase(it);
    }
    if (use().stream)
        (void)hipStreamSynchronize(use().stream);
    if (use().pool == b.pool)
        use().bytes -= (int64_t)b.size;
    if (!b.reusable) {
        std::shared_lock<std::shared_mutex> lk(release_mu());
        (void)hipFree(p);
    }
    {
        std::lock_guard<std::mutex> lk(b.pool->mu_);
        b.pool->out_ -= b.size;
        if (b.reusable) {
            b.pool->idle_.emplace(b.size, p);
            b.pool->idle_bytes_ += b.size;
        }
    }
    b.pool->trim(kMaxIdle);
    return true;
}

void DevPool::trim(size_t most)
{
    std::vector<void *> drop;
    {
        std::lock_guard<std::mutex> lk(mu_);
        const size_t keep = std::min({most, kMaxIdle, limit_ > out_ ? limit_ - out_ : (size_t)0});
        while (idle_bytes_ > keep) {  // the largest first
            auto it = std::prev(idle_.end());
            drop.push_back(it->second);
            idle_bytes_ -= it->first;
            idle_.erase(it);
        }
    }
    for (void *p : drop) {
        {
            std::lock_guard<std::mutex> lk(reg_mu());
            reg().erase(p);
        }
        std::shared_lock<std::shared_mutex> lk(release_mu());
        (void)hipFree(p);
    }
}

hipStream_t DevPool::take_stream()
{
    std::lock_guard<std::mutex> lk(mu_);
    if (streams_.empty())
        return nullptr;
    hipStream_t s = streams_.back();
    streams_.pop_back();
    return s;
}

bool DevPool::give_stream(hipStream_t s)
{
    std::lock_guard<std::mutex> lk(mu_);
    if (streams_.size() >= kMaxStreams)
        return false;
    streams_.push_back(s);
    return true;
}

}  // namespace ppcg
