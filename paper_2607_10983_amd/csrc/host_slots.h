// Slots of pinned host memory, kHostDoubles doubles each, one per context: a
// pinned allocation costs more than a small solve, so slots come from pages
// that are reused.  A page whose slots are all back is released, except one
// that is kept for the next context.  Safe with several threads.
#pragma once
#include <cstddef>
#include <mutex>
#include <vector>

namespace mg {

constexpr size_t kHostDoubles = 128, kPageSlots = 8;

class HostSlots {
public:
    typedef int (*Alloc)(double** page, size_t bytes);  // 0, or an error that take() returns
    typedef void (*Free)(double* page);

    HostSlots(Alloc a, Free f) : alloc_(a), free_(f) {}

    int take(double** out) {
        std::lock_guard<std::mutex> lock(m_);
        for (Page& p : pages_) {
            if (p.used == kFull) continue;
            size_t k = 0;
            while (p.used & (1u << k)) ++k;
            p.used |= 1u << k;
            *out = p.base + k * kHostDoubles;
            return 0;
        }
        pages_.reserve(pages_.size() + 1);
        double* base = nullptr;
        const int e = alloc_(&base, kPageSlots * kHostDoubles * sizeof(double));
        if (e != 0) return e;
        pages_.push_back(Page{base, 1u});
        *out = base;
        return 0;
    }

    void back(double* slot) {
        double* release = nullptr;
        {
            std::lock_guard<std::mutex> lock(m_);
            bool spare = false;
            size_t mine = pages_.size();
            for (size_t i = 0; i < pages_.size(); ++i) {
                Page& p = pages_[i];
                if (slot >= p.base && slot < p.base + kPageSlots * kHostDoubles) {
                    p.used &= ~(1u << (size_t)(slot - p.base) / kHostDoubles);
                    mine = i;
                } else if (p.used == 0) {
                    spare = true;
                }
            }
            if (spare && mine < pages_.size() && pages_[mine].used == 0) {
                release = pages_[mine].base;
                pages_.erase(pages_.begin() + mine);
            }
        }
        if (release) free_(release);
    }

private:
    struct Page {
        double* base;
        unsigned used;  // a bit per slot
    };
    static constexpr unsigned kFull = (1u << kPageSlots) - 1;
    Alloc alloc_;
    Free free_;
    std::mutex m_;
    std::vector<Page> pages_;
};

}  // namespace mg
