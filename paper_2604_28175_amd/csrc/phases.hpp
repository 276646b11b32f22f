// How a thread wants the batches that it submits to be run.
#pragma once

namespace strait {

// While a thread holds one of these, its batches are not begun before their input is complete (strait_submit begins a large staged one part by part).  The
// scheduling policy takes a batch for a transfer and then kernels (paper Eq. 1 to 3, 6): its profiles, and what the front end reports of each batch, have to be of such batches.
class InputFirst {
public:
    InputFirst() { ++held; }
    ~InputFirst() { --held; }
    InputFirst(const InputFirst&) = delete;
    InputFirst& operator=(const InputFirst&) = delete;
    static bool wanted() { return held > 0; }

private:
    inline static thread_local int held = 0;
};

}  // namespace strait
