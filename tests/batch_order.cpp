// Host-only check of the batch scheduler's stream ordering.  Linked with
// ns_batch.hip in place of the HIP runtime and the stage kernels: streams,
// events and captures are tracked as vector clocks, and every step of a member
// has to be ordered after the member's step before it, whatever streams the
// caller passes, which members come and go between calls, and whether steps run
// eagerly, from graphs or inside a capture of the caller's; and no graph may be
// destroyed before its last replay is known to have run.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <memory>
#include <random>
#include <set>
#include <vector>

#include "../paper_1709_09713_amd/csrc/ns_kernels.hpp"

namespace {

using Clock = std::map<int, long>;   // stream -> operations of it that are ordered before

struct Capture;
struct Stream {
    int id;
    Clock clk;                        // outside a capture, or within `cap`
    Capture *cap = nullptr;
    Clock before;                     // the clock outside, while in a capture
};
struct Event {
    Clock clk;
    Capture *cap = nullptr;
    bool recorded = false;
};
struct Step {
    int stream;
    long seq;
};
struct Capture {
    Stream *origin;
    std::set<Stream *> members;
    std::map<const void *, Step> last;   // of each state, in the capture
};
struct Graph {
    std::set<const void *> states;
    Step replay{0, 0};                   // the last one
};

int g_next = 1;
long g_seq = 0;
std::map<const void *, Step> g_last;
Clock g_done;                         // what the host knows to have run
std::mt19937 g_query(1);
int g_errors = 0;
const char *g_what = "";

Stream g_null{0};
Stream *str(hipStream_t s) { return s ? (Stream *)s : &g_null; }

void merge(Clock &a, const Clock &b)
{
    for (const auto &kv : b)
        if (a[kv.first] < kv.second) a[kv.first] = kv.second;
}

void fail(const char *msg)
{
    if (g_errors++ < 5) std::printf("%s: %s\n", g_what, msg);
}

// an operation on `state` in stream s
void operate(const void *state, Stream *s)
{
    auto &last = s->cap ? s->cap->last : g_last;
    auto it = last.find(state);
    if (it != last.end() && s->clk[it->second.stream] < it->second.seq)
        fail("a member's step is not ordered after its step before");
    const long q = ++g_seq;
    s->clk[s->id] = q;
    last[state] = Step{s->id, q};
}

}  // namespace

// ------------------------------------------------------------- HIP runtime
extern "C" {

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int)
{
    *s = (hipStream_t) new Stream{g_next++};
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete (Stream *)s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    merge(g_done, str(s)->clk);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e)
{
    if (g_query() % 2) return hipErrorNotReady;
    merge(g_done, ((Event *)e)->clk);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned int)
{
    *e = (hipEvent_t) new Event;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete (Event *)e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    Event *ev = (Event *)e;
    ev->clk = str(s)->clk;
    ev->cap = str(s)->cap;
    ev->recorded = true;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned int)
{
    Event *ev = (Event *)e;
    Stream *st = str(s);
    if (!ev->recorded) return hipSuccess;
    if (ev->cap != st->cap) {
        if (st->cap || st == &g_null) {
            fail("a stream under capture waits for an event from outside, or the reverse");
            return hipErrorStreamCaptureIsolation;
        }
        st->before = st->clk;
        st->clk.clear();
        st->cap = ev->cap;
        ev->cap->members.insert(st);
    }
    merge(st->clk, ev->clk);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    Stream *st = str(s);
    if (st->cap || st == &g_null) return hipErrorStreamCaptureUnsupported;
    st->before = st->clk;
    st->clk.clear();
    st->cap = new Capture{st, {st}, {}};
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    Stream *st = str(s);
    Capture *c = st->cap;
    if (!c || c->origin != st) return hipErrorStreamCaptureUnmatched;
    Graph *gr = new Graph;
    for (const auto &kv : c->last) {
        gr->states.insert(kv.first);
        if (st->clk[kv.second.stream] < kv.second.seq) fail("a captured step is not joined into the origin stream");
    }
    for (Stream *m : c->members) {
        m->clk = m->before;
        m->cap = nullptr;
    }
    delete c;
    *g = (hipGraph_t)gr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    *x = (hipGraphExec_t) new Graph(*(Graph *)g);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete (Graph *)g;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t g)
{
    const Step r = ((Graph *)g)->replay;
    if (g_done[r.stream] < r.seq) fail("a graph is destroyed before its replay has run");
    delete (Graph *)g;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t g, hipStream_t s)
{
    for (const void *state : ((Graph *)g)->states) operate(state, str(s));
    ((Graph *)g)->replay = Step{str(s)->id, g_seq};
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }

}  // extern "C"

// ------------------------------------------------------------- stage kernels
namespace ns {

ns_status make_fused_plan(const ns_params *p, ns_precision, int, int, double *state, void *, size_t, FusedPlan *out)
{
    *out = FusedPlan{};
    out->c.N = (int64_t)p->n[0] * p->n[1] * p->n[2];
    out->state = state;
    return NS_OK;
}

hipError_t enqueue_fused_step(const FusedPlan &f, double, ns_diag *diag, hipStream_t s)
{
    operate(f.state, str(s));
    if (diag) operate(diag, str(s));
    return hipSuccess;
}

}  // namespace ns

// -------------------------------------------------------------------- checks
namespace {

struct Run {
    ns_batch *b;
    char *memory;
    size_t at = 0;
    std::vector<hipStream_t> callers;
    explicit Run(int nstreams, int diag, int ncallers)
    {
        if (ns_batch_create(32, NS_FP64, nstreams, diag, &b) != NS_OK) std::abort();
        memory = (char *)((uintptr_t)1 << 40);   // addresses only; nothing is read or written
        for (int i = 0; i < ncallers; ++i) {
            hipStream_t s;
            hipStreamCreateWithFlags(&s, 0);
            callers.push_back(s);
        }
    }
    ~Run()
    {
        ns_batch_destroy(b);
        g_last.clear();
    }
    int add(int n, int steps)
    {
        ns_instance in = {};
        in.p.n[0] = in.p.n[1] = in.p.n[2] = n;
        in.dt = 1e-3;
        in.steps = steps;
        const size_t sb = 5 * (size_t)n * n * n * 8;
        in.state = (double *)(memory + at);
        in.work = memory + at + sb;
        in.work_bytes = 4 * sb;
        at += 5 * sb;
        int32_t slot = -1;
        if (ns_batch_add(b, &in, &slot) != NS_OK) return -1;
        return slot;
    }
    void step(int n, hipStream_t s)
    {
        if (ns_batch_step(b, n, (void *)s) != NS_OK) fail("ns_batch_step");
    }
};

// a large member ends, so that the one left changes stream
void two_members()
{
    g_what = "two members, two callers";
    Run r(2, 0, 2);
    r.add(64, 1);
    r.add(48, 9);
    r.step(1, r.callers[0]);
    r.step(1, r.callers[1]);
    r.step(3, r.callers[0]);
}

// the caller's stream under capture, after eager steps and twice in one capture
void caller_capture()
{
    g_what = "caller's capture";
    Run r(3, 1, 2);
    const int big = r.add(64, 100);
    r.add(48, 100);
    r.add(32, 100);
    r.step(2, r.callers[0]);
    ns_batch_remove(r.b, big);
    hipStreamBeginCapture(r.callers[1], hipStreamCaptureModeRelaxed);
    r.step(2, r.callers[1]);
    const int more = r.add(80, 100);
    r.step(1, r.callers[1]);
    ns_batch_remove(r.b, more);
    r.step(1, r.callers[1]);
    hipGraph_t g = nullptr;
    if (hipStreamEndCapture(r.callers[1], &g) != hipSuccess) fail("capture");
    hipGraphDestroy(g);
    r.step(2, r.callers[0]);
}

void random_calls(unsigned seed)
{
    g_what = "random calls";
    std::mt19937 rng(seed);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    Run r(pick(1, 8), pick(0, 1), pick(1, 3));
    std::vector<int> slots;
    for (int call = 0; call < 30; ++call) {
        if (pick(0, 2) == 0) ns_batch_set_graphs(r.b, pick(0, 1));
        for (int k = pick(0, 3); k > 0; --k) {
            const int s = r.add(8 * pick(1, 16), pick(1, 30));
            if (s >= 0) slots.push_back(s);
        }
        if (!slots.empty() && pick(0, 2) == 0) {
            const int i = pick(0, (int)slots.size() - 1);
            ns_batch_remove(r.b, slots[i]);
            slots.erase(slots.begin() + i);
        }
        r.step(pick(1, 20), pick(0, 4) == 0 ? nullptr : r.callers[pick(0, (int)r.callers.size() - 1)]);
    }
}

}  // namespace

int main()
{
    two_members();
    caller_capture();
    for (unsigned seed = 0; seed < 400; ++seed) random_calls(seed);
    std::printf("%d errors\n", g_errors);
    return g_errors != 0;
}
