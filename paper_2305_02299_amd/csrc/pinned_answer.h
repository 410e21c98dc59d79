// The wait for an answer that a launch writes into pinned host memory.  Host code that knows neither HIP nor Python, so that it can be compiled and
// tested by itself.
#pragma once
#include "srigl.h"

namespace srigl {

enum class StreamState { kBusy, kIdle, kUnknown };

// arrived(): whether the answer is complete.  state(): of the stream that the launch is on.  keep(): the memory must never be given back.
// The object stands between the memory and its return: it ends only when nothing can write there any more, however the calls went.
template <typename Arrived, typename State, typename Keep>
class PinnedAnswer {
public:
    PinnedAnswer(Arrived arrived, State state, Keep keep) : arrived_(arrived), state_(state), keep_(keep) {}
    PinnedAnswer(const PinnedAnswer&) = delete;
    PinnedAnswer& operator=(const PinnedAnswer&) = delete;
    ~PinnedAnswer() { wait(); }

    // Makes the call whose launch writes the answer.  The library refuses arguments and sizes before it launches anything; SRIGL_ERR_HIP is what it finds
    // behind the launch, which may be the error of an earlier call and the launch under way.
    template <typename Call>
    srigl_status launch(Call call) {
        pending_ = true;
        const srigl_status rc = call();
        if (rc != SRIGL_OK && rc != SRIGL_ERR_HIP) pending_ = false;
        return rc;
    }

    // Whether the answer has come.  Ends when it is there or the stream has finished without it; where the stream cannot say, the memory is kept.
    // (The stream is asked now and then only: asked every 1024 polls it took 6 us of a call's 22.)
    bool wait() {
        if (!pending_) return answered_;
        pending_ = false;
        for (unsigned polls = 1; !(answered_ = arrived_()); ++polls) {
            if (polls % 65536 != 0) continue;
            const StreamState s = state_();
            if (s == StreamState::kBusy) continue;
            answered_ = arrived_();
            if (s == StreamState::kUnknown && !answered_) keep_();
            break;
        }
        return answered_;
    }

private:
    Arrived arrived_;
    State state_;
    Keep keep_;
    bool pending_ = false, answered_ = false;
};

}  // namespace srigl
