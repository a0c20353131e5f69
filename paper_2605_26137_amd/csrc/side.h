// When a call of few faces may take the device's second stream (host code).
#pragma once

#include <mutex>

namespace bake {

// Bakes of few faces on several streams overlap each other better than their own
// two chains, which would all meet in the one second stream.  So a call takes it only
// when the kSteady calls before it on the device came from its own stream: streams
// that take turns, one call or several at a time, then never do.  Per bake at 5,120
// faces, 61,403 in brackets: four streams that take turns by twos 68 [92] us, two by
// eights 68 [136]; with only the one call before it asked for 83 [112] and 92 [167].
// One stream alone 112 [205], without the second stream 131 [220].
class SteadyCaller {
   public:
    static constexpr int kSteady = 16;

    // A call from `stream` (compared only); whether those before it were too.
    bool call(const void* stream) {
        std::lock_guard<std::mutex> lk(mu_);
        const bool steady = stream == last_ && run_ >= kSteady;
        run_ = stream == last_ ? (run_ < kSteady ? run_ + 1 : run_) : 1;
        last_ = stream;
        return steady;
    }

   private:
    std::mutex mu_;
    const void* last_ = nullptr;
    int run_ = 0;
};

}  // namespace bake
