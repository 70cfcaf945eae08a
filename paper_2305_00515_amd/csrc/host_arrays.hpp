// numpy arrays in host memory whose blocks are kept for the next ones: what a
// pipe hands out.  A new array of 2 MB costs its page faults on first use (the
// C library returns such a block to the system as soon as it is freed); a kept
// block does not.
//
// The blocks are ordinary memory, and each array owns its own (numpy's
// allocator interface, NEP 49): it can be resized, read by a forked process
// and dropped while somebody copies from it, as any array of numpy's.  (In
// page-locked memory it could not: the mapping is not inherited by a fork, and
// an asynchronous copy of the caller's may still read a block that is reused.)
// All of them come from malloc; the pool only puts off their free().  Blocks in
// use and idle together stay within the limit, beyond which arrays are plain
// ones.  The pool lives as long as the capsule and every array made with it;
// closing it frees the idle blocks, and later ones as they come back.
#pragma once

#include <numpy/arrayobject.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace {

struct HostPool {
    PyDataMem_Handler handler;
    std::mutex mu;
    std::unordered_map<size_t, std::vector<void *>> idle;   // by block size
    std::unordered_map<void *, size_t> used;                // blocks in arrays, with their size
    int64_t bytes = 0, limit = 0;                           // of all blocks; bound on them
    bool closed = false;
};

void *plain_block(size_t size)
{
    void *p = std::malloc(size);
    // as numpy does for its own arrays from 4 MB
    if (p && size >= (size_t)4 << 20) {
        const uintptr_t a = (reinterpret_cast<uintptr_t>(p) + 4095) & ~(uintptr_t)4095;
        madvise(reinterpret_cast<void *>(a), size - (a - reinterpret_cast<uintptr_t>(p)), MADV_HUGEPAGE);
    }
    return p;
}

// Frees idle blocks until `more` fits (all of them: more = limit + 1).
void pool_shrink(HostPool *h, int64_t more)
{
    for (auto &e : h->idle)
        while (h->bytes + more > h->limit && !e.second.empty()) {
            std::free(e.second.back());
            e.second.pop_back();
            h->bytes -= (int64_t)e.first;
        }
}

void *pool_malloc(void *ctx, size_t size)
{
    HostPool *h = static_cast<HostPool *>(ctx);
    size_t cap = 1;
    while (cap < size && cap) cap *= 2;
    try {
        std::lock_guard<std::mutex> lk(h->mu);
        std::vector<void *> &v = h->idle[cap];
        if (!v.empty()) {
            void *p = v.back();
            h->used.emplace(p, cap);
            v.pop_back();
            return p;
        }
        if (cap && (int64_t)cap <= h->limit) {
            pool_shrink(h, (int64_t)cap);
            if (h->bytes + (int64_t)cap <= h->limit)
                if (void *p = plain_block(cap)) {
                    try {
                        h->used.emplace(p, cap);
                    } catch (...) {
                        return p;   // a plain one
                    }
                    h->bytes += (int64_t)cap;
                    return p;
                }
        }
    } catch (...) {
    }
    return plain_block(size);
}

void *pool_calloc(void *, size_t n, size_t size) { return std::calloc(n, size); }

void pool_free(void *ctx, void *p, size_t)
{
    HostPool *h = static_cast<HostPool *>(ctx);
    {
        std::lock_guard<std::mutex> lk(h->mu);
        const auto it = h->used.find(p);
        if (it != h->used.end()) {
            const size_t cap = it->second;
            h->used.erase(it);
            if (!h->closed) {
                try {
                    h->idle[cap].push_back(p);
                    return;
                } catch (...) {
                }
            }
            h->bytes -= (int64_t)cap;
        }
    }
    std::free(p);
}

void *pool_realloc(void *ctx, void *p, size_t size)
{
    HostPool *h = static_cast<HostPool *>(ctx);
    {
        // no block of the pool's from here on
        std::lock_guard<std::mutex> lk(h->mu);
        const auto it = h->used.find(p);
        if (it != h->used.end()) {
            h->bytes -= (int64_t)it->second;
            h->used.erase(it);
        }
    }
    return std::realloc(p, size);
}

void pool_close(HostPool *h)
{
    std::lock_guard<std::mutex> lk(h->mu);
    h->closed = true;
    h->limit = 0;
    pool_shrink(h, h->bytes + 1);
}

constexpr const char *kPoolName = "mem_handler";   // what numpy asks of such a capsule

HostPool *pool_of(PyObject *capsule)
{
    auto *handler = static_cast<PyDataMem_Handler *>(PyCapsule_GetPointer(capsule, kPoolName));
    return handler ? static_cast<HostPool *>(handler->allocator.ctx) : nullptr;
}

void pool_delete(PyObject *capsule)
{
    if (HostPool *h = pool_of(capsule)) {   // no array is left: each held the capsule
        pool_close(h);
        delete h;
    }
}

// () -> a pool
PyObject *host_pool(PyObject *, PyObject *)
{
    HostPool *h = new (std::nothrow) HostPool;
    if (!h) return PyErr_NoMemory();
    std::memset(&h->handler, 0, sizeof h->handler);
    std::strcpy(h->handler.name, "sobel4x5_host_pool");
    h->handler.version = 1;
    h->handler.allocator = {h, pool_malloc, pool_calloc, pool_realloc, pool_free};
    PyObject *c = PyCapsule_New(&h->handler, kPoolName, pool_delete);
    if (!c) delete h;
    return c;
}

// (pool, height, width, limit in bytes) -> a new uint8 array
PyObject *host_array(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 4) return PyErr_Format(PyExc_TypeError, "expected 4 arguments, got %zd", n);
    HostPool *h = pool_of(a[0]);
    if (!h) return nullptr;
    npy_intp dims[2] = {PyLong_AsSsize_t(a[1]), PyLong_AsSsize_t(a[2])};
    const long long limit = PyLong_AsLongLong(a[3]);
    if (PyErr_Occurred()) return nullptr;
    {
        std::lock_guard<std::mutex> lk(h->mu);
        if (!h->closed) h->limit = limit;
    }
    PyObject *old = PyDataMem_SetHandler(a[0]);   // of this thread's context, for one array
    if (!old) return nullptr;
    PyObject *r = PyArray_SimpleNew(2, dims, NPY_UINT8);
    PyObject *type, *value, *trace;
    PyErr_Fetch(&type, &value, &trace);
    PyObject *back = PyDataMem_SetHandler(old);
    Py_DECREF(old);
    if (!back) {
        Py_CLEAR(r);
        Py_XDECREF(type);
        Py_XDECREF(value);
        Py_XDECREF(trace);
        return nullptr;
    }
    Py_DECREF(back);
    PyErr_Restore(type, value, trace);
    return r;
}

// (pool) -> bytes of its blocks, in use and idle
PyObject *host_bytes(PyObject *, PyObject *pool)
{
    HostPool *h = pool_of(pool);
    if (!h) return nullptr;
    std::lock_guard<std::mutex> lk(h->mu);
    return PyLong_FromLongLong(h->bytes);
}

// (pool): frees the idle blocks and keeps none from now on
PyObject *host_close(PyObject *, PyObject *pool)
{
    HostPool *h = pool_of(pool);
    if (!h) return nullptr;
    pool_close(h);
    Py_RETURN_NONE;
}

}  // namespace
