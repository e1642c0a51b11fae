// Arrays of a handle, cut from chunks of device memory (arena.hpp).
#include "arena.hpp"

#include <hip/hip_runtime_api.h>

#include <algorithm>

#include "ldu.h"

namespace ldu {

static void *try_alloc(size_t bytes) {
    void *p = nullptr;
    if (hipMalloc(&p, bytes) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}

// device memory for a request; where there is none, the chunks that lie free in
// the handle's pool go back first (their free waits for the device)
static void *device_alloc(size_t bytes, ChunkPool *pool) {
    void *p = try_alloc(bytes);
    if (!p && pool && pool->trim()) p = try_alloc(bytes);
    if (!p) throw Error(LDU_ERR_NOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
    return p;
}

// a chunk for a request of `bytes` beside `total` bytes held already: half as
// much again, at least 64 KiB (small matrices keep to what the runtime hands
// out of its own pages) and at most 512 MiB, or just the request when that
// much is not there
static Chunk new_chunk(size_t bytes, size_t total, ChunkPool *pool, bool grows = true) {
    Chunk c;
    if (!grows) total = 0;
    c.bytes = std::max(bytes, std::min(std::max(total / 2, size_t(64) << 10), size_t(512) << 20));
    void *p = c.bytes > bytes ? try_alloc(c.bytes) : nullptr;
    if (!p) {
        c.bytes = bytes;
        p = device_alloc(bytes, pool);
    }
    c.p = static_cast<char *>(p);
    return c;
}

Chunk ChunkPool::take(size_t bytes) {
    free_.reserve(free_.size() + out_ + 1);
    size_t best = free_.size();
    for (size_t k = 0; k < free_.size(); ++k)
        if (free_[k].bytes >= bytes && (best == free_.size() || free_[k].bytes < free_[best].bytes))
            best = k;
    if (best < free_.size()) {
        Chunk c = free_[best];
        c.used = 0;
        free_[best] = free_.back();
        free_.pop_back();
        ++out_;
        return c;
    }
    const Chunk c = new_chunk(bytes, total_, this);
    total_ += c.bytes;
    ++out_;
    return c;
}

bool ChunkPool::trim() {
    const bool any = !free_.empty();
    for (const Chunk &c : free_) {
        (void)hipFree(c.p);
        total_ -= c.bytes;
    }
    free_.clear();
    return any;
}

Arena::~Arena() { release_all(); }

// The last chunk, or else the fullest one that has room for `bytes`, or a new
// one: a large array that needs a chunk of its own leaves the rest of the others
// to later arrays.  The last chunk first keeps the arrays of a level together
// (CG + V-cycle at 100^3, fullest chunk first: 15.2 ms, last chunk first 15.0).
Chunk &Arena::chunk_for(size_t bytes) {
    if (!chunks_.empty() && chunks_.back().bytes - chunks_.back().used >= bytes)
        return chunks_.back();
    Chunk *best = nullptr;
    for (Chunk &c : chunks_)
        if (c.bytes - c.used >= bytes && (!best || c.bytes - c.used < best->bytes - best->used))
            best = &c;
    if (best) return *best;
    chunks_.reserve(chunks_.size() + 1);
    chunks_.push_back(temporary_ ? pool_->take(bytes) : new_chunk(bytes, total_, pool_, grows_));
    total_ += chunks_.back().bytes;
    return chunks_.back();
}

void Arena::check_denied() {
    if (pool_ && pool_->denied()) throw Error(LDU_ERR_NOMEM, "device array refused on request");
}

void *Arena::alloc(size_t bytes) {
    check_denied();
    bytes = (std::max(bytes, size_t(16)) + 255) & ~size_t(255);
    Chunk &c = chunk_for(bytes);
    void *p = c.p + c.used;
    c.used += bytes;
    return p;
}

void *Arena::alloc_own(size_t bytes) {
    check_denied();
    own_.reserve(own_.size() + 1);
    own_.push_back(device_alloc(std::max(bytes, size_t(16)), pool_));
    return own_.back();
}

void Arena::release(void *p) {
    for (size_t k = 0; k < own_.size(); ++k)
        if (own_[k] == p) {
            (void)hipFree(p);
            own_[k] = own_.back();
            own_.pop_back();
            return;
        }
}

Arena::Step::Step(Arena &a) : a_(&a) {
    for (const Chunk &c : a.chunks_) used_.push_back(c.used);
}

Arena::Step::~Step() {
    if (!a_) return;
    (void)hipDeviceSynchronize();  // the step's kernels may still write there
    for (; a_->chunks_.size() > used_.size(); a_->chunks_.pop_back()) {
        const Chunk &c = a_->chunks_.back();
        a_->total_ -= c.bytes;
        if (a_->temporary_) a_->pool_->put(c);
        else (void)hipFree(c.p);
    }
    for (size_t k = 0; k < used_.size(); ++k) a_->chunks_[k].used = used_[k];
}

void Arena::release_all() {
    for (const Chunk &c : chunks_) {
        if (temporary_) pool_->put(c);
        else (void)hipFree(c.p);
    }
    chunks_.clear();
    for (void *p : own_) (void)hipFree(p);
    own_.clear();
    total_ = 0;
}

}  // namespace ldu
