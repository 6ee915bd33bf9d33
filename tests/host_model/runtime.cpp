// Memory and threads of the CPU runtime (hip/hip_runtime.h).
#include "hip/hip_runtime.h"

#include <sys/mman.h>
#include <unistd.h>

#include <csignal>
#include <map>

namespace host {

HostGraph* capture = nullptr;
Index thread, block, block_dim, grid_dim;
static const char* running = "host code";

void stop(const char* what) {
    std::fprintf(stderr, "%s in %s, block (%u, %u, %u), thread (%u, %u)\n", what, running, block.x, block.y, block.z,
                 thread.x, thread.y);
    std::fflush(stderr);
    _exit(3);
}

// ---- memory -------------------------------------------------------------------
struct Area {
    char* map;
    size_t len, bytes;  // of the mapping, of the allocation
    char* p;
};
static std::map<void*, Area> areas;
static int side = 1;  // 1: the allocation ends at the mapping's end
constexpr unsigned char FILL = 0xff;  // a NaN in every format

static void on_fault(int, siginfo_t* si, void*) {
    char b[160];
    std::snprintf(b, sizeof b, "access out of range at %p", si->si_addr);
    for (auto& kv : areas) {
        const Area& a = kv.second;
        const char* at = (const char*)si->si_addr;
        if (at >= a.map - 4096 && at < a.map + a.len + 4096)
            std::snprintf(b, sizeof b, "access out of range, %ld bytes from the start of an allocation of %zu",
                          (long)(at - a.p), a.bytes);
    }
    stop(b);
}

void* guarded(size_t bytes) {
    const size_t page = 4096, len = (bytes + page - 1) / page * page + (bytes == 0 ? page : 0);
    char* m = (char*)mmap(nullptr, len + 2 * page, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED || mprotect(m + page, len, PROT_READ | PROT_WRITE)) stop("out of memory");
    m += page;
    std::memset(m, FILL, len);
    // allocations keep the alignment that the widest access needs
    char* p = side ? m + (len - bytes) / 16 * 16 : m;
    areas[p] = {m, len, bytes, p};
    return p;
}

static void check(const Area& a) {
    for (char* q = a.map; q < a.map + a.len; ++q)
        if ((q < a.p || q >= a.p + a.bytes) && (unsigned char)*q != FILL) stop("store beside an allocation");
}

void release(void* p) {
    if (!p) return;
    auto it = areas.find(p);
    if (it == areas.end()) stop("free of memory that is not allocated");
    check(it->second);
    munmap(it->second.map - 4096, it->second.len + 8192);
    areas.erase(it);
}

// LDS of one array of one kernel: NaN again when a block takes it first
static std::vector<void*> used;
void* block_lds(void*& cell, size_t bytes) {
    if (!cell) cell = guarded(bytes);
    for (void* u : used)
        if (u == cell) return cell;
    used.push_back(cell);
    std::memset(cell, FILL, bytes);
    return cell;
}

// ---- threads ------------------------------------------------------------------
// A fibre is its stack pointer; switch_to keeps the registers that a call keeps
// (x86-64) on the stack it leaves.
extern "C" void host_switch_to(void** from, void* to);
asm(R"(
.text
.globl host_switch_to
host_switch_to:
    push %rbp
    push %rbx
    push %r12
    push %r13
    push %r14
    push %r15
    mov %rsp, (%rdi)
    mov %rsi, %rsp
    pop %r15
    pop %r14
    pop %r13
    pop %r12
    pop %rbx
    pop %rbp
    ret
)");

struct Fibre {
    void* sp;
    bool done;
    Index id;
};
constexpr size_t STACK = 128 << 10;
constexpr int MAX_THREADS = 1024;
static char* stacks = nullptr;
static Fibre fibre[MAX_THREADS];
static void* scheduler;
static int current = 0, count = 0, descending = 0;
static const std::function<void()>* body = nullptr;
static double slot[MAX_THREADS];

void barrier() { host_switch_to(&fibre[current].sp, scheduler); }

static void entry() {
    (*body)();
    fibre[current].done = true;
    barrier();
}

double wave_xor(double v, int mask) {
    slot[current] = v;
    barrier();
    const int o = (current & ~63) | ((current & 63) ^ mask);
    const double r = o < count ? slot[o] : v;
    barrier();
    return r;
}

bool wave_any(bool v) {
    slot[current] = v;
    barrier();
    bool r = false;
    for (int l = current & ~63; l < count && l <= (current | 63); ++l) r = r || (!fibre[l].done && slot[l] != 0.0);
    barrier();
    return r;
}

static void run_block(dim3 b) {
    count = (int)(b.x * b.y * b.z);
    used.clear();
    for (int i = 0; i < count; ++i) {
        Fibre& f = fibre[i];
        f.done = false;
        f.id = {i % b.x, i / b.x % b.y, i / (b.x * b.y)};
        // six registers and the return address, the stack aligned as after a call
        void** top = (void**)(stacks + (size_t)(i + 1) * STACK) - 2;
        top[0] = (void*)entry;
        f.sp = top - 6;
    }
    for (int left = count; left > 0;) {
        left = 0;
        for (int k = 0; k < count; ++k) {
            current = descending ? count - 1 - k : k;
            if (fibre[current].done) continue;
            thread = fibre[current].id;
            host_switch_to(&scheduler, fibre[current].sp);
            left += !fibre[current].done;
        }
    }
}

static void run(const char* name, dim3 g, dim3 b, const std::function<void()>& f) {
    if (!stacks) {
        stacks = (char*)mmap(nullptr, MAX_THREADS * STACK, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        if (stacks == MAP_FAILED) stop("out of memory");
    }
    running = name;
    body = &f;
    block_dim = {b.x, b.y, b.z};
    grid_dim = {g.x, g.y, g.z};
    for (unsigned z = 0; z < g.z; ++z)
        for (unsigned y = 0; y < g.y; ++y)
            for (unsigned x = 0; x < g.x; ++x) {
                block = {x, y, z};
                run_block(b);
            }
    running = "host code";
}

void launch(const char* name, dim3 g, dim3 b, const std::function<void()>& f) {
    running = name;
    if (g.x == 0 || g.y == 0 || g.z == 0 || g.y > 65535 || g.z > 65535 || b.x * b.y * b.z == 0 ||
        b.x * b.y * b.z > MAX_THREADS)
        stop("launch outside the limits");
    if (capture)
        capture->nodes.push_back([=] { run(name, g, b, f); });
    else
        run(name, g, b, f);
}

}  // namespace host

extern "C" {
// allocations from now on end (1) or start (0) at an inaccessible page; order of a
// block's threads between two barriers; stores beside any allocation so far
void host_side(int s) { host::side = s; }
void host_order(int d) { host::descending = d; }
void host_check() {
    for (auto& kv : host::areas) host::check(kv.second);
}
void* host_malloc(size_t n) { return host::guarded(n); }
void host_free(void* p) { host::release(p); }
void host_begin() {
    static char alt[64 << 10];
    stack_t ss{};
    ss.ss_sp = alt;
    ss.ss_size = sizeof alt;
    sigaltstack(&ss, nullptr);
    struct sigaction sa {};
    sa.sa_sigaction = host::on_fault;
    sa.sa_flags = SA_SIGINFO | SA_ONSTACK;
    sigaction(SIGSEGV, &sa, nullptr);
    sigaction(SIGBUS, &sa, nullptr);
}
}
