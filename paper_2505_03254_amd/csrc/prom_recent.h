// What was computed for the last N keys, found again by the whole key.
#pragma once

namespace prom {

// The N keys used last (T: default-constructible; Key: trivially comparable by ==).  A program's blocks come in the
// same order again and again, so the search begins behind the entry found last and mostly ends there.
template <class Key, class T, int N> class Recent {
public:
    // The entry of `key`; *found tells whether it holds what was put there for this key, otherwise the caller fills it.
    T &get(const Key &key, bool *found)
    {
        int oldest = 0;
        for (int k = 1; k <= N; ++k) {
            const int i = (last_ + k) % N;
            if (used_[i] != 0 && keys_[i] == key) {
                *found = true;
                return touch(i);
            }
        }
        for (int i = 1; i < N; ++i)
            if (used_[i] < used_[oldest]) oldest = i;
        keys_[oldest] = key;
        *found = false;
        return touch(oldest);
    }

private:
    T &touch(int i)
    {
        used_[i] = ++clock_;
        last_ = i;
        return values_[i];
    }
    Key keys_[N] = {};
    T values_[N] = {};
    unsigned long long used_[N] = {}, clock_ = 0;  // 0: empty
    int last_ = N - 1;
};

}  // namespace prom
