// When a stack's frames are replayed from recorded graphs: while issuing a frame kernel by kernel takes the host longer
// than the GPU takes per frame.  Plain host code, no HIP.
#pragma once

namespace dc {

struct ReplayRule {
    bool on = false;
    float host_us = 0.f;        // issuing a frame kernel by kernel (running means; 0: nothing measured yet)
    float between_us = 0.f;     // what the caller spends between two calls
    float period_us = 0.f;      // distance of consecutive frames' ends on the GPU (a frame bound by the host shows the two about equal)

    static constexpr int kFirstFrames = 3;      // frames that pay for first uses (code objects, memory) are no measure
    static constexpr int kRefresh = 256;        // replayed frames after which one is issued kernel by kernel, to measure again (weighs as
                                                // much as what is known; it costs up to a frame's time: at 64, 1 to 2 % of a ResNet-50 stream)

    // A call that issued a frame kernel by kernel: `us` is its time without the waits in it (for a timed frame, a drain, a table).
    // idle: the frames before it were not all still running (or this one is a refresh).  A call that finds the GPU so
    // far behind is not what bounds it, and may have been held up by full queues.
    void issued(float us, bool idle) {
        ++frames;
        since_refresh = 0;
        if (frames > kFirstFrames && idle) mean(host_us, us, on ? 0.5f : 0.125f);
        decide();
    }
    void replayed() { ++frames; ++since_refresh; }
    bool refresh() const { return on && since_refresh >= kRefresh; }
    void between(float us) {
        if (us < 50.f) mean(between_us, us);
    }
    void period(float us) {     // a pause between frames is no measure of the GPU; eight in a row are no pauses
        if (period_us > 0.f && us > 2.f * period_us && ++gaps < 8) return;
        gaps = 0;
        mean(period_us, us);
        decide();
    }

private:
    int frames = 0, since_refresh = 0, gaps = 0;
    void mean(float& m, float us, float weight = 0.125f) { m = m > 0.f ? m + weight * (us - m) : us; }
    void decide() { on = host_us > 0.f && period_us > 0.f && host_us + between_us > (on ? 1.f : 0.97f) * period_us; }
};

}  // namespace dc
