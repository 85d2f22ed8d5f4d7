// Hardware lanes: user-mode queues of the GPU that mt_run fills with dispatch packets itself.
//
// A kernel launch through a HIP stream costs the host 2.5 to 3 us and the dependent launch after it starts 2.3 us after
// the previous one on an otherwise idle chip.  Both bound this library: a pass is a few hundred short kernels whose
// arguments do not change from run to run.  A packet written straight into a queue costs the host 0.03 us, and with
// agent-scope fences (what a kernel needs that reads what the kernel before it wrote) a dependent launch follows every
// 1.6 us (measured on MI355X, one-workgroup kernels, arguments in device memory).
//
// Queues of one process are dealt to the four dispatch pipes of the chip in the order of their creation, and two queues
// of one pipe take turns at about 7 us a turn: chains on two queues of different pipes take 1.8 us per launch of both,
// on the same pipe 14.4 us; four chains on four pipes 2.1 us, eight on eight queues 17 us.  A device therefore has four
// plain lanes, one per pipe, for the life of the process; a fifth tenant stream shares a lane (see lane_plan in
// runtime.cpp).  Streams restricted to a share of the compute units need queues of their own.
#pragma once
#include <hsa/hsa.h>
#include <hsa/hsa_ext_amd.h>

#include <atomic>
#include <list>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "internal.h"
#include "record.h"

namespace mt {

constexpr int N_LANES = 4;

// A queue packet: the 32-bit header goes last, with release order, when the packet is published.
struct alignas(64) Packet {
    uint32_t head;
    uint8_t body[60];
};

// Argument memory of one plan, in device memory the host can write.
struct KernargBlock {
    uint8_t *p = nullptr;
    size_t bytes = 0;
};

class LaneDevice {
public:
    // The lanes of HIP device `device`, opened on first use and kept for the life of the process; null with a
    // description in `why` if they cannot be opened.
    static LaneDevice *get(int device, std::string *why);

    hsa_queue_t *plain(int lane) const { return plain_[lane]; }
    // A queue restricted to the compute units of `mask`; null on failure.
    hsa_queue_t *create_masked(const std::vector<uint32_t> &mask);
    void destroy_queue(hsa_queue_t *q);

    const KernelCode *kernel(const void *host_fn);       // null if the kernel is not in this library's code objects
    uint8_t *static_scratch() const { return static_scratch_; }

    bool alloc_args(size_t bytes, KernargBlock *out);
    void free_args(KernargBlock b);
    hsa_signal_t take_signal();                          // handle 0 on failure
    void return_signal(hsa_signal_t s);

    // Publishes n packets and rings the doorbell.  False if the queue reported an error.
    bool submit(hsa_queue_t *q, const Packet *p, size_t n);
    // Waits until the signal has reached zero, polling.  False if a queue reported an error.
    bool wait(hsa_signal_t s);
    // Start and end of the dispatch a signal completed, in ms of one common clock.
    void times(hsa_signal_t s, double *start_ms, double *end_ms) const;
    bool failed() const { return error_.load(std::memory_order_relaxed) != 0; }

private:
    LaneDevice() = default;
    bool open(int device, std::string *why);
    bool load_code(std::string *why);
    static void queue_error(hsa_status_t s, hsa_queue_t *q, void *self);

    int device_ = 0;
    hsa_agent_t gpu_{};
    std::vector<hsa_agent_t> access_;                    // agents that touch argument memory: the GPU and the CPUs
    hsa_amd_memory_pool_t vram_{};
    double ms_per_tick_ = 0;
    uint8_t *static_scratch_ = nullptr;
    hsa_queue_t *plain_[N_LANES] = {};
    std::vector<hsa_executable_t> code_;
    // Held while packets are placed and the doorbell is rung.  Two queues may share one: what a queue waits for is always in its
    // queue already, so the holder never waits for another thread's packets.
    static constexpr int N_PRODUCERS = 16;
    std::mutex producer_[N_PRODUCERS];
    std::mutex mu_;                                      // kernels_, idle_signals_, the argument allocator
    std::unordered_map<const void *, std::unique_ptr<KernelCode>> kernels_;
    std::vector<hsa_signal_t> idle_signals_;
    std::map<uint8_t *, size_t> free_args_;              // free pieces of the argument chunks, by address
    std::atomic<int> error_{0};
};

// Header word of a kernel dispatch packet.  barrier: starts after every packet before it has completed.
inline uint32_t dispatch_head(bool barrier, int acquire, int release, int dims) {
    return (uint32_t)(HSA_PACKET_TYPE_KERNEL_DISPATCH << HSA_PACKET_HEADER_TYPE) | ((barrier ? 1u : 0u) << HSA_PACKET_HEADER_BARRIER) |
           ((uint32_t)acquire << HSA_PACKET_HEADER_SCACQUIRE_FENCE_SCOPE) | ((uint32_t)release << HSA_PACKET_HEADER_SCRELEASE_FENCE_SCOPE) |
           ((uint32_t)dims << (16 + HSA_KERNEL_DISPATCH_PACKET_SETUP_DIMENSIONS));
}
Packet dispatch_packet(const RecordedLaunch &l, void *kernarg, uint32_t head, hsa_signal_t done);
Packet wait_packet(const hsa_signal_t *deps, int n);     // nothing after it starts before the (at most 5) signals are zero
// Writes a launch's arguments, explicit and implicit, at `dst` (l.code->kernarg_bytes bytes).
void write_args(const RecordedLaunch &l, const uint8_t *explicit_args, uint8_t *dst);
void publish_args(const uint8_t *last_byte);             // argument memory written so far is visible to packets published next

}  // namespace mt
