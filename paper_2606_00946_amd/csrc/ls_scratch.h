// Scratch layouts of the data path's calls (ls_buffer_push, ls_train_round).
// Host code, no HIP.
//
// A layout is written once, as the carving itself: with no buffer behind it the
// same function gives the bytes to allocate, so a size can not differ from what
// is taken.
#pragma once

#include <cstddef>
#include <cstdint>

namespace ls {

inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

struct WsCarve {
    char* base = nullptr;
    size_t cap = SIZE_MAX;   // bytes behind base
    size_t off = 0;
    template <class T>
    T* take(int64_t count) {
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off += (size_t)round_up(count * (int64_t)sizeof(T), 256);
        return p;
    }
    bool ok() const { return off <= cap; }
};

// One push of B rows: nc of them or of the FIFO's become candidates, n_all rows
// (pool and candidates) go through the forward.
struct PushScratch {
    int32_t* codes;          // [nc + B]
    float *cx, *cy;          // candidate rows
    float *ax, *ay;          // forward input
    float* forward;
    double* cemb;            // candidate embeddings
    int32_t* admitted;       // count, where the caller wants none
    char* admission;
};

inline PushScratch carve_push(WsCarve& w, int32_t B, int32_t nc, int32_t n_all, int d, int H, int64_t forward_floats,
                              int64_t admission_bytes) {
    PushScratch s;
    s.codes = w.take<int32_t>((int64_t)nc + B);
    s.cx = w.take<float>((int64_t)nc * d);
    s.cy = w.take<float>(nc);
    s.ax = w.take<float>((int64_t)n_all * d);
    s.ay = w.take<float>(n_all);
    s.forward = w.take<float>(forward_floats);
    s.cemb = w.take<double>((int64_t)nc * H);
    s.admitted = w.take<int32_t>(1);
    s.admission = w.take<char>(admission_bytes);
    return s;
}

// A round of `epochs` passes over n rows in minibatches of `batch`.
struct TrainScratch {
    int32_t* codes;          // [epochs x n]
    float *bx, *by;          // one minibatch's rows
    float* step_loss;
    double* loss_sum;
    char* update;
};

inline TrainScratch carve_train(WsCarve& w, int32_t epochs, int32_t n, int32_t batch, int d, int64_t update_bytes) {
    TrainScratch s;
    s.codes = w.take<int32_t>((int64_t)epochs * n);
    s.bx = w.take<float>((int64_t)batch * d);
    s.by = w.take<float>(batch);
    s.step_loss = w.take<float>(1);
    s.loss_sum = w.take<double>(1);
    s.update = w.take<char>(update_bytes);
    return s;
}

}  // namespace ls
