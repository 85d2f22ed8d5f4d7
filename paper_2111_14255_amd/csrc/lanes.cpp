// Hardware lanes (see lanes.h): the library's code objects loaded a second time through the HSA loader, so that kernels
// can be named in dispatch packets, and the queues, signals and argument memory those packets use.
#include "lanes.h"

#include <link.h>
#include <sched.h>

#include <algorithm>
#include <cstdio>
#include <cstring>

namespace mt {

namespace {

constexpr uint32_t QUEUE_PACKETS = 4096;
constexpr size_t ARG_ALIGN = 256, ARG_CHUNK = (size_t)1 << 20;

inline void pause_once() {
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
}

thread_local LaunchRecorder *recorder_of_thread = nullptr;

// The read-only segments of this library in memory.
std::vector<std::pair<const uint8_t *, size_t>> own_segments() {
    static const char here = 0;
    struct Find {
        uintptr_t inside;
        std::vector<std::pair<const uint8_t *, size_t>> found;
    } f{(uintptr_t)&here, {}};
    (void)dl_iterate_phdr([](dl_phdr_info *o, size_t, void *u) {
        Find *f = (Find *)u;
        std::vector<std::pair<const uint8_t *, size_t>> segs;
        bool own = false;
        for (int i = 0; i < o->dlpi_phnum; ++i) {
            const ElfW(Phdr) &h = o->dlpi_phdr[i];
            if (h.p_type != PT_LOAD) continue;
            const uintptr_t at = (uintptr_t)(o->dlpi_addr + h.p_vaddr);
            own = own || (f->inside >= at && f->inside < at + h.p_memsz);
            if ((h.p_flags & PF_R) && !(h.p_flags & PF_W)) segs.push_back({(const uint8_t *)at, (size_t)h.p_filesz});
        }
        if (own) f->found = std::move(segs);
        return own ? 1 : 0;
    }, &f);
    return f.found;
}

// The gfx950 code objects inside the loaded library: one offload bundle per device source, each a table of (offset, size,
// target) followed by the objects.  They are read from memory, where they stay while the library is loaded; its file may have
// been replaced or removed since.
std::vector<std::pair<const uint8_t *, size_t>> own_code_objects() {
    std::vector<std::pair<const uint8_t *, size_t>> out;
    for (auto [base, size] : own_segments()) {
        for (size_t at = (8 - (uintptr_t)base % 8) % 8; at + 64 < size;) {
            // the magic in two parts, so that the segment holds it in bundles only
            if (std::memcmp(base + at, "__CLANG_OFFL", 12) != 0 || std::memcmp(base + at + 12, "OAD_BUNDLE__", 12) != 0) { at += 8; continue; }
            const size_t left = size - at;
            uint64_t count = 0;
            std::memcpy(&count, base + at + 24, 8);
            size_t pos = 32, end = 32;
            for (uint64_t e = 0; e < count && pos + 24 <= left; ++e) {
                uint64_t h[3];                           // offset, size, length of the target name
                std::memcpy(h, base + at + pos, 24);
                if (h[2] > left - pos - 24) break;
                const std::string target((const char *)base + at + pos + 24, (size_t)h[2]);
                pos += 24 + (size_t)h[2];
                if (h[0] <= left && h[1] <= left - h[0]) {
                    end = std::max<size_t>(end, (size_t)(h[0] + h[1]));
                    if (h[1] > 0 && target.find("gfx950") != std::string::npos) out.push_back({base + at + h[0], (size_t)h[1]});
                }
            }
            at += (std::max(end, pos) + 7) / 8 * 8;
        }
    }
    return out;
}

}  // namespace

LaunchRecorder *&current_recorder() { return recorder_of_thread; }

void LaunchRecorder::add(const void *host_fn, dim3 grid, dim3 block, size_t lds, const void *packed, size_t bytes) {
    const KernelCode *code = dev->kernel(host_fn);
    if (!code || bytes > code->kernarg_bytes) {
        if (!error) error = (int)hipErrorInvalidDeviceFunction;
        return;
    }
    RecordedLaunch l{code, {grid.x, grid.y, grid.z}, {block.x, block.y, block.z}, (uint32_t)lds, args.size(), bytes};
    args.insert(args.end(), (const uint8_t *)packed, (const uint8_t *)packed + bytes);
    launches.push_back(l);
}

// ---- device ---------------------------------------------------------------------------------------
LaneDevice *LaneDevice::get(int device, std::string *why) {
    static std::mutex mu;
    static std::map<int, LaneDevice *> open_devices;     // never destroyed: queues live as long as the process
    std::lock_guard<std::mutex> lk(mu);
    auto it = open_devices.find(device);
    if (it != open_devices.end()) return it->second;
    std::unique_ptr<LaneDevice> d(new LaneDevice);
    if (!d->open(device, why)) return nullptr;
    return open_devices[device] = d.release();
}

void LaneDevice::queue_error(hsa_status_t s, hsa_queue_t *, void *self) {
    ((LaneDevice *)self)->error_.store(s == HSA_STATUS_SUCCESS ? -1 : (int)s);
}

bool LaneDevice::open(int device, std::string *why) {
    auto no = [&](const char *what) { if (why) *why = what; return false; };
    device_ = device;
    int bus = 0, dev = 0, domain = 0;
    if (hipDeviceGetAttribute(&bus, hipDeviceAttributePciBusId, device) != hipSuccess ||
        hipDeviceGetAttribute(&dev, hipDeviceAttributePciDeviceId, device) != hipSuccess ||
        hipDeviceGetAttribute(&domain, hipDeviceAttributePciDomainId, device) != hipSuccess)
        return no("the device has no PCI address");
    if (hsa_init() != HSA_STATUS_SUCCESS) return no("hsa_init failed");
    struct Find { uint32_t bdf, domain; hsa_agent_t gpu{}; std::vector<hsa_agent_t> cpus; } f{(uint32_t)(bus << 8 | dev << 3), (uint32_t)domain, {}, {}};
    (void)hsa_iterate_agents([](hsa_agent_t a, void *u) {
        Find *f = (Find *)u;
        hsa_device_type_t t;
        if (hsa_agent_get_info(a, HSA_AGENT_INFO_DEVICE, &t) != HSA_STATUS_SUCCESS) return HSA_STATUS_SUCCESS;
        if (t == HSA_DEVICE_TYPE_CPU) f->cpus.push_back(a);
        uint32_t bdf = 0, dom = 0;
        if (t == HSA_DEVICE_TYPE_GPU && hsa_agent_get_info(a, (hsa_agent_info_t)HSA_AMD_AGENT_INFO_BDFID, &bdf) == HSA_STATUS_SUCCESS &&
            hsa_agent_get_info(a, (hsa_agent_info_t)HSA_AMD_AGENT_INFO_DOMAIN, &dom) == HSA_STATUS_SUCCESS && (bdf & ~7u) == f->bdf && dom == f->domain)
            f->gpu = a;
        return HSA_STATUS_SUCCESS;
    }, &f);
    if (!f.gpu.handle) return no("no agent at the device's PCI address");
    gpu_ = f.gpu;
    access_ = f.cpus;
    access_.push_back(gpu_);
    (void)hsa_amd_agent_iterate_memory_pools(gpu_, [](hsa_amd_memory_pool_t p, void *u) {
        hsa_amd_segment_t seg;
        uint32_t flags = 0;
        if (hsa_amd_memory_pool_get_info(p, HSA_AMD_MEMORY_POOL_INFO_SEGMENT, &seg) == HSA_STATUS_SUCCESS && seg == HSA_AMD_SEGMENT_GLOBAL &&
            hsa_amd_memory_pool_get_info(p, HSA_AMD_MEMORY_POOL_INFO_GLOBAL_FLAGS, &flags) == HSA_STATUS_SUCCESS &&
            (flags & HSA_AMD_MEMORY_POOL_GLOBAL_FLAG_COARSE_GRAINED)) {
            *(hsa_amd_memory_pool_t *)u = p;
            return HSA_STATUS_INFO_BREAK;
        }
        return HSA_STATUS_SUCCESS;
    }, &vram_);
    if (!vram_.handle) return no("no device memory pool");
    uint64_t freq = 0;
    if (hsa_system_get_info(HSA_SYSTEM_INFO_TIMESTAMP_FREQUENCY, &freq) != HSA_STATUS_SUCCESS || freq == 0) return no("no timestamp frequency");
    ms_per_tick_ = 1e3 / (double)freq;
    if (!load_code(why)) return false;
    // four queues in a row: one per dispatch pipe
    for (int i = 0; i < N_LANES; ++i) {
        if (hsa_queue_create(gpu_, QUEUE_PACKETS, HSA_QUEUE_TYPE_MULTI, queue_error, this, UINT32_MAX, UINT32_MAX, &plain_[i]) != HSA_STATUS_SUCCESS)
            return no("a hardware queue could not be created");
        (void)hsa_amd_profiling_set_profiler_enabled(plain_[i], 1);
    }
    return true;
}

bool LaneDevice::load_code(std::string *why) {
    for (auto &o : own_code_objects()) {
        hsa_code_object_reader_t r;
        hsa_executable_t x;
        if (hsa_code_object_reader_create_from_memory(o.first, o.second, &r) != HSA_STATUS_SUCCESS ||
            hsa_executable_create_alt(HSA_PROFILE_FULL, HSA_DEFAULT_FLOAT_ROUNDING_MODE_DEFAULT, nullptr, &x) != HSA_STATUS_SUCCESS ||
            hsa_executable_load_agent_code_object(x, gpu_, r, nullptr, nullptr) != HSA_STATUS_SUCCESS ||
            hsa_executable_freeze(x, nullptr) != HSA_STATUS_SUCCESS) {
            if (why) *why = "a code object of the library could not be loaded";
            return false;
        }
        code_.push_back(x);
    }
    for (hsa_executable_t x : code_) {
        hsa_executable_symbol_t s;
        uint64_t at = 0;
        if (hsa_executable_get_symbol_by_name(x, STATIC_SCRATCH_SYMBOL, &gpu_, &s) == HSA_STATUS_SUCCESS &&
            hsa_executable_symbol_get_info(s, HSA_EXECUTABLE_SYMBOL_INFO_VARIABLE_ADDRESS, &at) == HSA_STATUS_SUCCESS)
            static_scratch_ = (uint8_t *)at;
    }
    if (!static_scratch_ && why) *why = code_.empty() ? "no gfx950 code object found in the library" : "the fixed scratch array is not in the code objects";
    return static_scratch_ != nullptr;
}

const KernelCode *LaneDevice::kernel(const void *host_fn) {
    std::lock_guard<std::mutex> lk(mu_);
    auto it = kernels_.find(host_fn);
    if (it != kernels_.end()) return it->second.get();
    std::unique_ptr<KernelCode> k;
    const char *name = hipKernelNameRefByPtr(host_fn, nullptr);
    for (size_t i = 0; name && !k && i < code_.size(); ++i) {
        hsa_executable_symbol_t s;
        if (hsa_executable_get_symbol_by_name(code_[i], (std::string(name) + ".kd").c_str(), &gpu_, &s) != HSA_STATUS_SUCCESS) continue;
        k.reset(new KernelCode);
        if (hsa_executable_symbol_get_info(s, HSA_EXECUTABLE_SYMBOL_INFO_KERNEL_OBJECT, &k->object) != HSA_STATUS_SUCCESS ||
            hsa_executable_symbol_get_info(s, HSA_EXECUTABLE_SYMBOL_INFO_KERNEL_KERNARG_SEGMENT_SIZE, &k->kernarg_bytes) != HSA_STATUS_SUCCESS ||
            hsa_executable_symbol_get_info(s, HSA_EXECUTABLE_SYMBOL_INFO_KERNEL_GROUP_SEGMENT_SIZE, &k->group_bytes) != HSA_STATUS_SUCCESS ||
            hsa_executable_symbol_get_info(s, HSA_EXECUTABLE_SYMBOL_INFO_KERNEL_PRIVATE_SEGMENT_SIZE, &k->private_bytes) != HSA_STATUS_SUCCESS)
            k.reset();
    }
    return (kernels_[host_fn] = std::move(k)).get();
}

hsa_queue_t *LaneDevice::create_masked(const std::vector<uint32_t> &mask) {
    hsa_queue_t *q = nullptr;
    if (hsa_queue_create(gpu_, QUEUE_PACKETS, HSA_QUEUE_TYPE_MULTI, queue_error, this, UINT32_MAX, UINT32_MAX, &q) != HSA_STATUS_SUCCESS) return nullptr;
    (void)hsa_amd_profiling_set_profiler_enabled(q, 1);
    const hsa_status_t s = hsa_amd_queue_cu_set_mask(q, (uint32_t)mask.size() * 32, mask.data());
    if (s != HSA_STATUS_SUCCESS && s != (hsa_status_t)HSA_STATUS_CU_MASK_REDUCED) {
        (void)hsa_queue_destroy(q);
        return nullptr;
    }
    return q;
}

void LaneDevice::destroy_queue(hsa_queue_t *q) {
    if (q) (void)hsa_queue_destroy(q);
}

// ---- argument memory: first fit over free pieces, neighbours joined again when a piece is returned -------------
bool LaneDevice::alloc_args(size_t bytes, KernargBlock *out) {
    bytes = (std::max<size_t>(bytes, 1) + ARG_ALIGN - 1) / ARG_ALIGN * ARG_ALIGN;
    std::lock_guard<std::mutex> lk(mu_);
    for (int attempt = 0; attempt < 2; ++attempt) {
        for (auto it = free_args_.begin(); it != free_args_.end(); ++it) {
            if (it->second < bytes) continue;
            uint8_t *p = it->first;
            const size_t rest = it->second - bytes;
            free_args_.erase(it);
            if (rest) free_args_[p + bytes] = rest;
            *out = KernargBlock{p, bytes};
            return true;
        }
        const size_t chunk = (bytes + ARG_CHUNK - 1) / ARG_CHUNK * ARG_CHUNK;
        void *p = nullptr;
        if (hsa_amd_memory_pool_allocate(vram_, chunk, 0, &p) != HSA_STATUS_SUCCESS) return false;
        if (hsa_amd_agents_allow_access((uint32_t)access_.size(), access_.data(), nullptr, p) != HSA_STATUS_SUCCESS) {
            (void)hsa_amd_memory_pool_free(p);
            return false;
        }
        free_args_[(uint8_t *)p] = chunk;
    }
    return false;
}

void LaneDevice::free_args(KernargBlock b) {
    if (!b.p) return;
    std::lock_guard<std::mutex> lk(mu_);
    auto it = free_args_.emplace(b.p, b.bytes).first;
    auto next = std::next(it);
    if (next != free_args_.end() && it->first + it->second == next->first) {
        it->second += next->second;
        free_args_.erase(next);
    }
    if (it != free_args_.begin()) {
        auto prev = std::prev(it);
        if (prev->first + prev->second == it->first) {
            prev->second += it->second;
            free_args_.erase(it);
        }
    }
}

hsa_signal_t LaneDevice::take_signal() {
    {
        std::lock_guard<std::mutex> lk(mu_);
        if (!idle_signals_.empty()) {
            hsa_signal_t s = idle_signals_.back();
            idle_signals_.pop_back();
            return s;
        }
    }
    hsa_signal_t s{0};
    // no interrupt on completion: the host polls
    if (hsa_amd_signal_create(1, 0, nullptr, HSA_AMD_SIGNAL_AMD_GPU_ONLY, &s) != HSA_STATUS_SUCCESS) s.handle = 0;
    return s;
}

void LaneDevice::return_signal(hsa_signal_t s) {
    if (!s.handle) return;
    std::lock_guard<std::mutex> lk(mu_);
    idle_signals_.push_back(s);
}

// ---- packets --------------------------------------------------------------------------------------
bool LaneDevice::submit(hsa_queue_t *q, const Packet *p, size_t n) {
    // one producer at a time: the doorbell has to rise with the packets, whichever thread rings it
    std::lock_guard<std::mutex> lk(producer_[((uintptr_t)q >> 6) % N_PRODUCERS]);
    while (n > 0) {
        const size_t part = std::min<size_t>(n, q->size / 2);
        const uint64_t at = hsa_queue_add_write_index_relaxed(q, part);
        while (at + part - hsa_queue_load_read_index_scacquire(q) > q->size) {
            if (failed()) return false;
            pause_once();
        }
        Packet *ring = (Packet *)q->base_address;
        const uint64_t wrap = q->size - 1;
        for (size_t i = 0; i < part; ++i) std::memcpy(ring[(at + i) & wrap].body, p[i].body, sizeof(p[i].body));
        for (size_t i = 0; i < part; ++i) __atomic_store_n(&ring[(at + i) & wrap].head, p[i].head, __ATOMIC_RELEASE);
        hsa_signal_store_screlease(q->doorbell_signal, (hsa_signal_value_t)(at + part - 1));
        p += part;
        n -= part;
    }
    return !failed();
}

bool LaneDevice::wait(hsa_signal_t s) {
    for (uint64_t spins = 1; hsa_signal_load_scacquire(s) > 0; ++spins) {
        if ((spins & 1023) == 0 && failed()) return false;
        if (spins < 1000000) pause_once();
        else sched_yield();                              // tens of milliseconds: leave the core to others now and then
    }
    return !failed();
}

void LaneDevice::times(hsa_signal_t s, double *start_ms, double *end_ms) const {
    hsa_amd_profiling_dispatch_time_t t{};
    (void)hsa_amd_profiling_get_dispatch_time(gpu_, s, &t);
    *start_ms = (double)t.start * ms_per_tick_;
    *end_ms = (double)t.end * ms_per_tick_;
}

Packet dispatch_packet(const RecordedLaunch &l, void *kernarg, uint32_t head, hsa_signal_t done) {
    hsa_kernel_dispatch_packet_t k{};
    k.workgroup_size_x = (uint16_t)l.block[0];
    k.workgroup_size_y = (uint16_t)l.block[1];
    k.workgroup_size_z = (uint16_t)l.block[2];
    k.grid_size_x = l.grid[0] * l.block[0];
    k.grid_size_y = l.grid[1] * l.block[1];
    k.grid_size_z = l.grid[2] * l.block[2];
    k.private_segment_size = l.code->private_bytes;
    k.group_segment_size = l.code->group_bytes + l.dyn_lds;
    k.kernel_object = l.code->object;
    k.kernarg_address = kernarg;
    k.completion_signal = done;
    Packet p;
    static_assert(sizeof(p) == sizeof(k), "packets are 64 bytes");
    std::memcpy(&p, &k, sizeof(p));
    p.head = head;
    return p;
}

Packet wait_packet(const hsa_signal_t *deps, int n) {
    hsa_barrier_and_packet_t b{};
    for (int i = 0; i < n; ++i) b.dep_signal[i] = deps[i];
    Packet p;
    static_assert(sizeof(p) == sizeof(b), "packets are 64 bytes");
    std::memcpy(&p, &b, sizeof(p));
    p.head = (uint32_t)(HSA_PACKET_TYPE_BARRIER_AND << HSA_PACKET_HEADER_TYPE) | (1u << HSA_PACKET_HEADER_BARRIER);
    return p;
}

// Implicit arguments follow the explicit ones, 8-byte aligned, in the order the compiler documents for code objects of
// version 5: workgroup counts (3 x 4 bytes), workgroup sizes (3 x 2), remainders (3 x 2, zero: whole workgroups only),
// ... dimensions at 64, dynamic LDS at 120.
void write_args(const RecordedLaunch &l, const uint8_t *explicit_args, uint8_t *dst) {
    const size_t n = l.code->kernarg_bytes, base = (l.arg_bytes + 7) / 8 * 8;
    alignas(16) uint8_t buf[4096];
    uint8_t *out = n <= sizeof(buf) ? buf : dst;
    std::memset(out, 0, n);
    std::memcpy(out, explicit_args, l.arg_bytes);
    auto put = [&](size_t off, auto v) {
        if (base + off + sizeof(v) <= n) std::memcpy(out + base + off, &v, sizeof(v));
    };
    int dims = 3;
    if (l.grid[2] * l.block[2] == 1) dims = l.grid[1] * l.block[1] == 1 ? 1 : 2;
    for (int i = 0; i < 3; ++i) put(4 * (size_t)i, l.grid[i]);
    for (int i = 0; i < 3; ++i) put(12 + 2 * (size_t)i, (uint16_t)l.block[i]);
    put(64, (uint16_t)dims);
    put(120, l.dyn_lds);
    if (out == buf) std::memcpy(dst, buf, n);
}

// Host writes to device memory are posted and may sit in write-combining buffers: the fence drains those, and a read of
// what was written last returns only when the writes before it have arrived.
void publish_args(const uint8_t *last_byte) {
#if defined(__x86_64__)
    __builtin_ia32_sfence();
#endif
    (void)*(const volatile uint8_t *)last_byte;
    std::atomic_thread_fence(std::memory_order_seq_cst);
}

}  // namespace mt
