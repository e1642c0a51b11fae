// Device memory of a handle: arrays cut from chunks, and the chunks that the
// temporary arrays of one call hand on to each other.  Host code only.
#pragma once

#include <cstddef>
#include <cstdint>
#include <stdexcept>
#include <string>
#include <vector>

namespace ldu {

struct Error : std::runtime_error {
    int code;
    Error(int c, const std::string &m) : std::runtime_error(m), code(c) {}
};

// Device memory comes in chunks that several arrays share: a call of hipMalloc
// or hipFree for more than a few megabytes takes 0.1-0.3 ms whatever its size,
// and setup makes hundreds of arrays.  Matrix, hierarchy and first solve of a
// 121x117x130 mesh: 115 -> 84 ms (2 ms of that from the solve).
struct Chunk {
    char *p = nullptr;
    size_t bytes = 0, used = 0;
};

// chunks that a handle's temporary arenas hand on to each other during one
// call.  A handle runs one call on one stream at a time, so a reused chunk is
// ordered behind its last use by that stream; trim() gives the free ones back at
// the end of the call, and when a request does not fit beside them (whether
// there were any).
class ChunkPool {
public:
    ~ChunkPool() { trim(); }
    Chunk take(size_t bytes);
    // called from destructors: take() has made the room it needs
    void put(Chunk c) noexcept {
        free_.push_back(c);
        --out_;
    }
    bool trim();
    // whether the array asked for now is refused (ldu_deny_memory)
    bool denied() { return ++asked && deny > 0 && --deny == 0; }
    int64_t asked = 0, deny = 0;

private:
    std::vector<Chunk> free_;
    size_t total_ = 0, out_ = 0;  // bytes of all chunks; chunks with an arena
};

class Arena {  // owns device memory: a handle's, a hierarchy's, or one step's
public:
    Arena() = default;
    explicit Arena(ChunkPool *pool) : pool_(pool), temporary_(true) {}
    // a temporary arena over the same pool as `like`
    explicit Arena(const Arena *like) : pool_(like->pool_), temporary_(like->pool_ != nullptr) {}
    Arena(const Arena &) = delete;
    Arena &operator=(const Arena &) = delete;
    ~Arena();
    void use_pool(ChunkPool *pool) { pool_ = pool; }  // for the temporaries made from this one
    void *alloc(size_t bytes);
    // an array of its own, for release()
    void *alloc_own(size_t bytes);
    template <typename T>
    T *get(size_t count) { return static_cast<T *>(alloc(count * sizeof(T))); }
    // room for `bytes` more in one chunk
    void reserve(size_t bytes) { (void)chunk_for(bytes); }
    // chunks of the requests' own size from now on: what is still to come are
    // single sets of arrays, not the hundreds of a set-up
    void settle() { grows_ = false; }
    void release(void *p);  // frees one alloc_own allocation of this arena
    void release_all();

    // what is cut from an arena after this, given back when the step that asked
    // for it does not come to done()
    class Step {
    public:
        explicit Step(Arena &a);
        ~Step();
        Step(const Step &) = delete;
        Step &operator=(const Step &) = delete;
        void done() { a_ = nullptr; }

    private:
        Arena *a_;
        std::vector<size_t> used_;
    };

private:
    Chunk &chunk_for(size_t bytes);
    void check_denied();
    std::vector<Chunk> chunks_;
    std::vector<void *> own_;
    size_t total_ = 0;  // bytes of all chunks
    ChunkPool *pool_ = nullptr;
    bool temporary_ = false, grows_ = true;
};

}  // namespace ldu
